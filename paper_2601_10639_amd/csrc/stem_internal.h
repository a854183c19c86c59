// Internal declarations shared by libstem's translation units (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/stem.h"

typedef uint16_t bf16_t;  // raw bfloat16 bits

// ---- kernel ids for the profiling table -----------------------------------------
enum StemKernelId {
  K_GEMM_GATE = 0,   // G = X Wg^T with fused SiLU*gather epilogue
  K_GEMM_GATE_PLAIN, // G = X Wg^T, plain store (host-resident table mode)
  K_GEMM_DOWN,       // Y = H Wd^T
  K_GEMM_DH,         // dH = dY Wd with fused dU/dG epilogue
  K_GEMM_DX,         // dX = dG Wg
  K_GEMM_DWDOWN,     // dWd = dY^T H
  K_GEMM_DWGATE,     // dWg = dG^T X
  K_SILU_GATHER,     // H = SiLU(G) * E[ids] (stand-alone)
  K_SORT_COUNT,
  K_SORT_SCAN,
  K_SORT_SCATTER,
  K_SORT_FUSED,
  K_UNIQUE,
  K_SEG_REDUCE,
  K_SEG_COMBINE,
  K_ADAMW,
  K_ROW_COPY,        // host-resident rows -> compact device table
  K_SPLITK_REDUCE,   // sum of split-K partial products
  K_GEMM_UP,         // Up = X Wu^T (dense SwiGLU and the additive variant)
  K_GEMM_DWUP,       // dWu = dV^T X
  K_SORT_MERGE,
  K_GRADS_F32,       // dx, dWd and dWg of a small fp32 layer in one launch
  K_GEMM_DW,         // two or three weight gradients in one launch
  K_LIST_COPY,       // host-resident table: remap and the row copy's lists
  K_FFN_DECODE,      // a decode step's layer in one launch
  K_COUNT_
};

#define STEM_MAX_PROF_EVENTS 8192
#define STEM_PF_MAX_CHUNKS 16
#define STEM_EDIT_MAX_TOKENS 64
// 256x256 down-product tiles per chunk of a host-table batch: one round on the compute units that a row copy leaves free, with
// room to spare (prefetch.hip).  65536 tokens of 2048 x 8192, ms, calls in turn on two contexts / by itself: 256 tiles 4.88 / 4.89
// with a copy stream per context, 240 tiles 4.97 / 4.69 and 4.13 / 4.59 with one for all, 224 tiles 4.60 / 4.70 and 4.11 / 4.64; 16384
// tokens 240 tiles 1.42 / 1.74, 224 tiles 1.42 / 1.69; 1024 x 4096, 16384 tokens 0.652 / 0.870 and 0.648 / 0.843.
#define STEM_PF_CHUNK_TILES 224
// Bytes of rows from which a host-table call is long (api.hip): it takes the first copy stream, and the others the second meanwhile
#define STEM_PF_LONG ((int64_t)128 << 20)

struct stem_ctx {
  stem_layer_desc desc;
  int64_t max_tokens;
  int device;
  char err[512];

  // scratch, all device memory unless noted
  void* H_ws;            // [max_tokens, F] context dtype
  void* dG_ws;           // [max_tokens, F] context dtype
  void* Up_ws;           // [max_tokens, F] bf16, allocated by the first stem_ffn_up_* call
  float* splitk_ws;      // fp32 partial products of GEMMs whose K range is cut into slices
  size_t splitk_bytes;   // its size; no launch splits beyond it
  int32_t* tickets;      // [STEM_TICKETS] counters of finished K slices per output tile, zero between launches
  unsigned long long* rounds; // [STEM_TICKETS] the same for the few-row kernel, which counts on from launch to launch
  uint32_t* sync;        // [33 * 256] flags, 32 times, and claims of the layer in one launch (ffn_decode_bf16.hip)
  int polls;             // how often a workgroup of the few-row kernel looks for the others
  int looks;             // and of the layer in one launch
  int two_launches;      // a layer that one launch would do takes two (tests)
  int32_t* sort_keys[2]; // [max_tokens]
  int32_t* sort_vals[2]; // [max_tokens]
  int32_t* sort_counts;  // [64 * waves]
  int32_t* seg_of;       // [max_tokens] index of the segment each sorted position is in
  int64_t seg_T;         // T of the call that last wrote seg_of (-1 = none)
  float* seg_part;       // [chunks][2][F] partial sums of segments that cross chunk borders
  int32_t* flag;         // pinned host int, device-visible: sticky id-range flag

  // host-resident table mode
  hipStream_t side;      // the one of the device's two copy streams that the last prefetch took
  hipEvent_t ready;      // rows and remap of the last prefetch are there
  hipEvent_t promoted;   // and the rows it has put into the cache are copied too
  hipEvent_t done;       // the one of these two that is behind all copies of the last prefetch
  int copies_open;       // a prefetch has put copies on the side stream and not recorded that event
  int32_t* slot;         // host [V], -1 = absent
  int32_t* uniq_pinned;  // pinned host [max_tokens]
  int32_t* remap_pinned; // pinned host [max_tokens]
  int32_t* uniq_dev;     // device [max_tokens]
  int32_t* order_pinned; // pinned host [2 * max_tokens]: table row, then compact slot, in order of first use
  int32_t* order_dev;    // device [2 * max_tokens]
  // chunks of the last prefetch: tokens [k * pf_chunk_tokens, ...) need only rows copied before pf_ev[k]
  int pf_chunks;         // 0 = the last prefetch recorded no per-chunk events
  int64_t pf_T, pf_chunk_tokens;
  hipEvent_t pf_ev[STEM_PF_MAX_CHUNKS];
  int prefetch_mode;     // STEM_PREFETCH_KERNEL or STEM_PREFETCH_MEMCPY
  char* pack_pinned;     // pinned host staging for the memcpy mode
  size_t pack_bytes;
  hipEvent_t pack_done[2];

  // device-resident cache of hot rows in host-resident mode (host-side bookkeeping; the rows
  // themselves live in the caller's buffer)
  int64_t cache_slots;       // 0 = no cache
  int32_t* cache_id_in_slot; // host [cache_slots], -1 = free
  int32_t* cache_slot_of;    // host [V], -1 = not cached
  uint32_t* cache_freq;      // host [V]: token occurrences seen so far
  int32_t* inst_pinned;      // pinned host [2 * max_tokens]: promoted rows (staging row, then cache slot)
  int32_t* inst_dev;         // device [2 * max_tokens]

  // knowledge editing: device scratch for up to STEM_EDIT_MAX_TOKENS source / target tokens
  int32_t* edit_idx_dev;     // [3 * STEM_EDIT_MAX_TOKENS]: source rows, picked rows, target rows
  void* edit_rep_dev;        // [STEM_EDIT_MAX_TOKENS, F] replacement rows

  // profiling
  int prof_on;
  hipEvent_t* prof_ev;   // 2 * STEM_MAX_PROF_EVENTS
  int prof_kid[STEM_MAX_PROF_EVENTS];
  int prof_n;
  double prof_ms[K_COUNT_];
  int64_t prof_launches[K_COUNT_];
};

// Brackets a launch with events when profiling is on.
struct ProfScope {
  stem_ctx* c;
  hipStream_t s;
  int idx;
  ProfScope(stem_ctx* ctx, int kid, hipStream_t st) : c(ctx), s(st), idx(-1) {
    if (c && c->prof_on && c->prof_n < STEM_MAX_PROF_EVENTS) {
      idx = c->prof_n++;
      c->prof_kid[idx] = kid;
      (void)hipEventRecord(c->prof_ev[2 * idx], s);
    }
  }
  ~ProfScope() {
    if (idx >= 0) (void)hipEventRecord(c->prof_ev[2 * idx + 1], s);
  }
};

// ---- bf16 MFMA GEMM family (gemm_bf16.hip) ---------------------------------------
// C[m,n] = sum_k Aop[m,k] * Bop[n,k].  An operand is "KC" when stored [rows, K] with K
// contiguous, "MC" when stored [K, rows] with rows contiguous.
enum { OP_KC = 0, OP_MC = 1 };
enum GemmEpilogue {
  EPI_BF16 = 0, // C -> bf16 [M,N]
  EPI_F32,      // C -> fp32 [M,N], optional +=
  EPI_GATE,     // G (optional) and H = SiLU(C) * E[ids[m], n], both bf16
  EPI_DH,       // dU = C * SiLU(G), dG = C * E[ids[m], n] * SiLU'(G), both bf16
  EPI_SPLITK,   // decode kernel only: EPI_BF16 of a product in K slices
  // dense SwiGLU (UP) and the additive variant (UPE): SiLU(C) is multiplied by Up or Up + E[ids]
  EPI_GATE_UP, EPI_GATE_UPE,
  EPI_DH_UP, EPI_DH_UPE,
  EPI_BF16_RES, // C + residual -> bf16 [M,N] (decode chains: the layer's output joins the residual stream)
  EPI_GATE_DUAL, EPI_GATE_DUALE  // EPI_GATE_UP, EPI_GATE_UPE with Up computed beside C, in the same launch
};

struct GemmArgs {
  const bf16_t* A; // M-side operand
  const bf16_t* B; // N-side operand
  int M, N, K;
  int lda, ldb;    // leading dimensions of the stored operands
  void* C;         // EPI_BF16 / EPI_F32 output, ld = N
  const bf16_t* residual;  // EPI_BF16_RES (and the few-row kernel when not null): [M,N] bf16 added in fp32 before rounding
  // What one kernel has and others have not shares its place: every launch copies the whole block.
  union {
    int accumulate;  // EPI_F32: add to C
    int next_bytes;  // EPI_GATE in the decode and few-row kernels: how many bytes of `next` to bring closer (stem_touch_bytes)
    int polls;       // EPI_BF16 in the few-row kernel: the context's
  };
  const int32_t* ids;
  const bf16_t* E;
  int E_rows;
  bf16_t* outG;    // EPI_GATE: may be null
  bf16_t* outH;    // EPI_GATE
  union {
    const bf16_t* inUp; // *_UP, *_UPE: the up projection x W_up^T, [M,N] bf16
    bf16_t* outUp;      // *_DUAL*: where it goes
  };
  const bf16_t* A2;  // optional second operand pair of a (KC,KC) product: C = A B^T + A2 B2^T
  const bf16_t* B2;
  int K2;
  union {
    const bf16_t* inG;  // EPI_DH
    const bf16_t* Bup;  // *_DUAL*: W_up, as B
    const bf16_t* next; // EPI_GATE in the decode and few-row kernels: the weights of the product behind it
  };
  bf16_t* outdU;   // EPI_DH
  bf16_t* outdG;   // EPI_DH
  int32_t* flag;
  // room for split-K launches, null = never split.  fp32 partial products: [ksplit][M][N] of the large kernel; whole tiles,
  // [ksplit][tiles][...], of the decode and the few-row kernel (128x64), which is more where M or N is ragged
  float* ws;
  size_t ws_bytes; // capacity of ws
  union {
    int32_t* tickets;           // decode kernel: the context's tickets; null = never split
    unsigned long long* rounds; // few-row kernel: the context's rounds; null = never split
  };
  // Further products of the same K in the launch (weight gradients only, stem_weight_grads)
  struct { const bf16_t* A; const bf16_t* B; void* C; int M, N, lda, ldb; } more[2];
  int n_more;
  int64_t elems;   // outputs of all of the launch's products, filled in by the launcher
  int ksplit;      // number of k slices, chosen by the launcher
  int kc_skip;     // set by the large kernel itself: elements a K slice starts after the operand's start
  int mt, nt;      // few-row and decode kernels: tile counts and exact float reciprocals, filled in by the launcher
  float inv_mt, inv_per_z;
};

hipError_t stem_gemm_bf16(stem_ctx* ctx, int kid, int la, int lb, int epi, const GemmArgs& a, hipStream_t s);
// n = 2 or 3 weight gradients of a layer (both operands OP_MC, EPI_F32) in one launch: whether that is the shorter way, and the launch
struct GroupPlan { int tiling, ksplit; };
bool stem_weight_grads_together(const GemmArgs* a, int n, GroupPlan* plan);
hipError_t stem_weight_grads(stem_ctx* ctx, const GemmArgs* a, int n, const GroupPlan& plan, hipStream_t s);

// ---- which kernel a call takes, as its launcher decides it: exported for the tests, not part of stem.h ----
enum StemRoute { ROUTE_DECODE = 0, ROUTE_FEW_ROW, ROUTE_TILES };
extern "C" {
// route: {StemRoute, tile rows, tile columns, K slices}.  epi: GemmEpilogue; ops: operand pairs
void stem_route_tiles(int M, int N, int K, int ops, int epi, int64_t ws_bytes, int32_t* route);
// the n = 2 (dW_down, dW_gate) or 3 (dW_up too) weight gradients of a layer: {one launch, tile rows, tile columns, K slices}
void stem_route_weight_grads(int d_model, int d_ff, int64_t T, int n, int64_t ws_bytes, int32_t* route);
// workgroup `block` of a tile launch of n products of M x N outputs: {product, K slice, tile row, tile column}; returns the grid
int stem_route_tile(const int32_t* M, const int32_t* N, int n, int tile_rows, int tile_cols, int band, int ksplit, int block, int32_t* at);
// whether the weight gradients may share a launch before dx (null: not wanted) as their buffers lie; W_up, dV, dW_up: null without an up projection
int stem_route_weight_grads_apart(int d_model, int d_ff, int64_t T, const void* dy, const void* H, const void* dx, const void* W_gate,
                                  const void* W_up, const void* dV, const float* dW_gate, const float* dW_up);
// whether stem_ffn_up_forward's gate and up product may share a launch as the buffers lie (E, ids, G may be null)
int stem_route_gate_up_together(int d_model, int d_ff, int64_t T, const void* W_up, const void* E, int64_t E_rows, const void* ids,
                                const void* G, const void* Up, const void* H);
void stem_route_decode(int M, int N, int K, int epi, int64_t ws_bytes, int32_t* route);
// the gate (route[0..3]) and down (route[4..7]) products of a bf16 stem_ffn_forward call of T tokens that is not one launch, in a context made for
// as many
void stem_route_forward(int d_model, int d_ff, int64_t T, int32_t* route);
// whether a forward call with the table on the device is one launch (ffn_decode_bf16.hip): by size, and as its buffers lie (null: not there)
int stem_route_one_launch(int d_model, int d_ff, int64_t T);
int stem_route_one_launch_apart(int d_model, int d_ff, int64_t T, const void* G, const void* H, const void* W_down, const void* residual,
                                const void* y);
int64_t stem_route_splitk_bytes(int d_model, int d_ff, int64_t max_tokens);   // a context's room for K slices
int stem_route_sort(int64_t T, int V);   // SortRoute
// whether ranks by counting sort them: up to 2048 ids, where the vocabulary allows it and no two of the call's buffers overlap
int stem_route_sort_ranks(int64_t T, int V, const int32_t* ids, const int32_t* sorted_ids, const int32_t* perm, const int32_t* uniq_ids,
                          const int32_t* seg_offsets, const int32_t* n_uniq, const int32_t* seg_of);
// whether buckets of the vocabulary do: 2049 to 16384 ids, likewise
int stem_route_sort_buckets(int64_t T, int V, const int32_t* ids, const int32_t* sorted_ids, const int32_t* perm, const int32_t* uniq_ids,
                            const int32_t* seg_offsets, const int32_t* n_uniq, const int32_t* seg_of);
// whether the sort and the sums of a call with these buffers (dU may be null: no sums) are one launch
int stem_route_sort_sum(int is_bf16, int64_t T, int V, int F, const int32_t* ids, const void* dU, const int32_t* sorted_ids,
                        const int32_t* perm, const int32_t* uniq_ids, const int32_t* seg_offsets, const int32_t* n_uniq,
                        const int32_t* seg_of, const float* dE_rows);
int stem_route_touch_bytes(int d_model, int d_ff, int64_t T);   // of W_down, touched by the gate product of that call
// How many copy streams host-table calls of T tokens and this many distinct rows take in turn.  With one the link stands still between two
// calls' rows, and a copy that waits for compute units finds them taken by tiles (15 to 60 us a call); two hold 32 compute units
// instead of 16, and where products weigh as much as the rows, that and the later first rows cost more.  The line: 15 kFLOP of products
// per byte of rows (bf16 products of 1 PFLOP/s then take three quarters of the rows' time; the fp32 ones run at a thirteenth of that), and up
// to 1024 tokens layers of 12 M weights a matrix, whose products are one round on all compute units.  Calls in turn on three contexts, us, a
// stream for each / one / two in turn: 512 x 1536, 2000 tokens 52 / 65 / 55; 1024 x 4096, 2000 tokens 144 / 144 / 136, 8192 tokens 386 /
// 374 / 354, 65536 tokens (12 kFLOP a byte) 1727 / 1691 / 1643; 1536 x 5120, 2000 tokens 175 / 175 / 157, 49152 tokens (14.7) 2154 / 1978 / 1954;
// 2048 x 8192, 4096 tokens 495 / 470 / 453, 16384 tokens (14.4) 1462 / 1404 / 1357; against 1472 x 5248, vocabulary 8499, 12668 tokens (15.4)
// 591 / 495 / 515; 2048 x 8192, vocabulary 30000, 16384 tokens (17.6) 1360 / 1170 / 1240, 65536 tokens (20.3) 5234 / 4138 / 4862, 700 tokens 147 /
// 124 / 146; fp32, 256 x 1024, 8192 tokens (0.9) 212 / 203 / 197, 512 x 2048, vocabulary 8000, 2000 tokens (1.5) 156 / 131 / 149.  On two contexts two in
// turn are within 1 % of a stream for each, and of one but at 8192 tokens of 1024 x 4096 (381 / 393) and 4096 of 2048 x 8192 (470 / 510).
int stem_route_copy_streams(int d_model, int d_ff, int dtype, int64_t T, int64_t rows);
void stem_exchange_two_launches(stem_ctx* c, int on);   // no layer in one launch on this context
uint32_t stem_next_launch(uint32_t last);           // stem_launch_after, and
int stem_exchange_launch(stem_ctx* c, uint32_t last);   // all flags of the layer in one launch as launch `last` left them (waits for the device)
void stem_exchange_polls(stem_ctx* c, int polls);   // 0: no workgroup of the few-row kernel's K slices or of the layer in one launch waits for another
}
// By size, where stem_route_sort_ranks and stem_route_sort_buckets say no.
enum SortRoute { SORT_ONE_1024 = 0, SORT_ONE_4096, SORT_RUNS_1024, SORT_RUNS_4096, SORT_DIGITS };

// Bytes of W_down that the gate product of a decode-sized call touches, a dword per 128-byte line behind its first K tiles, so that
// the down product finds them in the memory-side cache: all or none.  L2 serves hits and misses in turn, so what the touches cost
// the gate product is what they save the down product in misses, and they pay where that one waits for its misses besides: from
// 112 tokens (below, the gate product waits for them itself) and 8 MB of weights (below, the launches are latency) to 16 MB, or 34
// up to 128 tokens, where the down product is the decode kernel's (above, the gate product is bound by L2).  Layer forward, us,
// without / with: 1024 x 4096, 112 tokens 16.9 / 16.7, 192 tokens 22.4 / 20.7, 384 tokens 27.7 / 26.0; 1280 x 5120, 128 tokens 28.0 /
// 25.3; 1536 x 5120, 384 tokens 41.2 / 37.4; 2048 x 8192, 128 tokens 35.3 / 34.3; against 1024 x 4096, 24
// tokens 12.4 / 13.4; 896 x 3584, 128 tokens 15.0 / 15.6; 2048 x 8192, 192 tokens 37.7 / 40.0; 1792 x 7168, 192 tokens 34.4 / 36.0; 128
// tokens of 2304 x 8192 42.6 / 45.7, of 2048 x 10240 47.7 / 51.5.
inline int stem_touch_bytes(int M, int d, int F) {
  const int64_t w = (int64_t)d * F * 2;
  return M >= 112 && M <= 512 && w >= 7900000 && w <= (M <= 128 ? 34 : 16) * 1000000ll ? (int)w : 0;
}

// ---- few-row bf16 GEMM (gemm_skinny_bf16.hip): both operands K-contiguous, K % 64 == 0 --------
// 128x64 tiles; used when M is small enough that larger tiles would leave most of the chip idle: up to 256 rows, and up
// to 512 while the gate product is one round of its workgroups.  Layer forward, us, this / 128x128 tiles: d_model 2048,
// d_ff 8192, 256 tokens 41 / 44, 320 tokens 59 / 48, 512 tokens 69 / 56; 1536 x 5120, 384 tokens 37.3 / 42.9, 512 tokens 55 / 44;
// 1024 x 4096, 320 tokens 26 / 28, 512 tokens 26 / 34.
bool stem_gemm_skinny_fits(int M, int F);
#define STEM_SPLITK_WS_MAX ((size_t)64 << 20)   // more is never worth it: beyond it the tiles fill the chip
// out = bf16(sum of the ksplit fp32 partial products in ws, in slice order (+ residual)); total elements each
hipError_t stem_splitk_reduce(stem_ctx* ctx, const float* ws, int ksplit, int64_t total, const bf16_t* residual, void* out,
                              hipStream_t s);
// k slices that bring the launch to about one workgroup per compute unit (1 = no split)
int stem_gemm_skinny_ksplit(int M, int N, int K, size_t ws_bytes);
// epi: EPI_BF16 (+ residual; split along K through a.ws and a.rounds) or EPI_GATE
hipError_t stem_gemm_skinny_bf16(stem_ctx* ctx, int kid, int epi, const GemmArgs& a, hipStream_t s);

// ---- decode-sized bf16 GEMM (gemm_decode_bf16.hip): both operands K-contiguous --------------------
#define STEM_TICKETS 256
#define STEM_COUNTERS (STEM_TICKETS * (8 + 4) + 33 * 256 * 4)   // bytes of a context's rounds, tickets, flags and claims
#define STEM_LOOKS 200    // some 100 us: the workgroups of a layer in one launch are some us apart unless other streams hold the compute units
#define STEM_POLLS 2000   // 1 to 2 ms: the slices of a tile are some us apart unless other streams hold the compute units
bool stem_gemm_decode_fits(int M, int N, int K);
// epi: EPI_BF16 (+ residual; split along K through a.ws and a.tickets where that pays) or EPI_GATE
hipError_t stem_gemm_decode_bf16(stem_ctx* ctx, int kid, int epi, const GemmArgs& a, hipStream_t s);

// ---- a decode step's layer in one launch (ffn_decode_bf16.hip): the table on the device ----
struct StemDecodeArgs {
  const bf16_t *x, *Wg, *Wd, *E, *residual;   // residual may be null
  const int32_t* ids;
  bf16_t *y, *save_G, *save_H;                // the saved ones may be null
  int T, d, F, E_rows;
};
hipError_t stem_ffn_decode_bf16(stem_ctx* ctx, const StemDecodeArgs& a, hipStream_t s);
// The number of the launch that finds its flags at `last`: never 0, which in a claim says that nothing was given up, and which would come
// again with every 2^32-th launch (6 to 18 hours of decoding on one context).  Numbers are compared for equality only.
__host__ __device__ inline uint32_t stem_launch_after(uint32_t last) { return last == 0xffffffffu ? 1u : last + 1u; }

// ---- fp32 path and element-wise kernels (kernels_f32.hip) -------------------------
struct GemmF32Args {
  const float* A; // M-side operand, leading dimension lda
  const float* B; // N-side operand
  int64_t lda, ldb;
  int M, N, K;
  float* C;          // EPI_F32: output; EPI_GATE: G, may be null; ld = N
  const float* add;  // EPI_F32: added to the product (C itself to accumulate, a residual), may be null
  const int32_t* ids;
  const float* E;
  int E_rows;
  const float* inG;  // EPI_DH
  float* out0;       // EPI_GATE: H; EPI_DH: dU
  float* out1;       // EPI_DH: dG
  int32_t* flag;
};
// operand kinds and epilogues (EPI_F32, EPI_GATE, EPI_DH) as for the bf16 products
hipError_t stem_gemm_f32(stem_ctx* ctx, int kid, int la, int lb, int epi, const GemmF32Args& p, hipStream_t s);
// dx (may be null), dW_down and dW_gate in one launch, where all three are small
bool stem_grads_f32_fits(const GemmF32Args* dx, const GemmF32Args& w0, const GemmF32Args& w1);
hipError_t stem_grads_f32(stem_ctx* ctx, const GemmF32Args* dx, const GemmF32Args& w0, const GemmF32Args& w1, hipStream_t s);
hipError_t stem_fill_zero(void* p, size_t bytes, hipStream_t s);   // a kernel, not a memset node
// H = SiLU(G) * E[ids]; is_bf16 selects the element type of G, E, H
hipError_t stem_silu_gather(stem_ctx* ctx, int is_bf16, const void* G, const int32_t* ids, const void* E,
                            int E_rows, void* H, int64_t T, int F, hipStream_t s);

// ---- table gradient (embed_grad.hip) ----------------------------------------------
// Device scratch of the sort and the segmented sum: a context's own buffers, or pieces of the
// library's static scratch array (the entry point that allocates nothing).
struct EmbedScratch {
  int32_t* sort_keys[2]; // [T] each (multi-kernel sort only)
  int32_t* sort_vals[2]; // [T] each
  int32_t* sort_counts;  // [stem_sort_count_entries(T)]
  int32_t* seg_of;       // [T] index of the run each sorted position is in
  float* seg_part;       // [stem_seg_chunks(T)][2][F] partial sums of runs that cross chunk borders
  int32_t* flag;         // sticky id-range flag (host-pinned or device)
};
hipError_t stem_sort_unique(stem_ctx* prof, const EmbedScratch& ws, const int32_t* ids, int64_t T, int V,
                            int32_t* sorted_ids, int32_t* perm, int32_t* uniq_ids, int32_t* seg_offsets,
                            int32_t* n_uniq, hipStream_t s);
hipError_t stem_seg_reduce(stem_ctx* prof, const EmbedScratch& ws, int is_bf16, const void* dU, const int32_t* perm,
                           const int32_t* seg_offsets, int64_t T, int F, float* dE_rows, hipStream_t s);
// both, or without dU the sort alone
hipError_t stem_table_grad(stem_ctx* prof, const EmbedScratch& ws, int is_bf16, const int32_t* ids, const void* dU, int64_t T, int V, int F,
                           int32_t* sorted_ids, int32_t* perm, int32_t* uniq_ids, int32_t* seg_offsets, int32_t* n_uniq, float* dE_rows,
                           hipStream_t s);
int64_t stem_seg_chunks(int64_t max_tokens);
int64_t stem_sort_count_entries(int64_t max_tokens);
// error text for calls that have no context (stem_last_error(NULL) returns it)
stem_status stem_fail(stem_ctx* c, stem_status st, const char* fmt, ...);

// ---- optimiser (adamw.hip) ----------------------------------------------------------
hipError_t stem_adamw(stem_ctx* ctx, int is_bf16, const int32_t* uniq_ids, const int32_t* n_uniq,
                      int64_t max_rows, const float* g, void* E, float* master, float* m, float* v, int F,
                      const stem_adamw_hparams& hp, hipStream_t s);

// ---- host-resident rows (prefetch.hip) ----------------------------------------------
// From pinned host memory to the device: remap [T], and entries [0, n) and [second, second + n) of order
hipError_t stem_copy_lists_kernel(stem_ctx* ctx, const int32_t* remap_host, int32_t* remap, int64_t T, const int32_t* order_host,
                                  int32_t* order, int64_t n, int64_t second, hipStream_t s);
// E_compact[dst_slot[k]] = E_host[src_row[k]] for k in [0, n)
hipError_t stem_copy_rows_kernel(stem_ctx* ctx, const void* E_host, const int32_t* src_row, const int32_t* dst_slot,
                                 int64_t n, int64_t row_bytes, void* E_compact, hipStream_t s);

// ---- knowledge editing (edit.hip) ----------------------------------------------------------
// rows E[src[j]] <- (pick[j] >= 0 ? old E[pick[j]] : mean of the old rows E[tgt[0..n_t)]); the old
// source rows go to backup (may be null).  rep: [n_s, F] scratch in the table's dtype.
hipError_t stem_edit_launch(stem_ctx* ctx, int is_bf16, void* E, const int32_t* src_dev, const int32_t* pick_dev,
                            const int32_t* tgt_dev, int n_s, int n_t, int F, void* rep, void* backup, hipStream_t s);
