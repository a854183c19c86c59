// A decode step's whole layer in one launch: y = (SiLU(x W_gate^T) * E[ids]) W_down^T [+ residual], up to 32 tokens, bf16, gfx950.
//
// Two launches of so few tokens are latency and weight bytes: each pays for its start (1.5 us), for the first bytes from HBM (1), for a
// reduction and for its end.  A workgroup here has 1 / 256 of either weight matrix in registers: W_gate's loads and half of W_down's are
// requested before anything waits, the other half behind the stores of H.  It computes its columns of H, publishes them, waits until
// every workgroup has done so, and multiplies all of H with its rows of W_down, of which it needs no K slices.
//
// Operands.  Weights go straight into MFMA fragments: 8 rows x 128 bytes a load, whole lines, as the fragment's 16 rows are the 8 rows
// at either of two neighbouring chunks of 8 k.  The tokens' fragments are 8 tokens at either chunk likewise, and of a 16 x 16 product
// the half counts in which both are at the same one.  Neighbouring lanes read 32 contiguous bytes then; with the two halves of a line as
// the two chunks they read 16, which cost 0.5 to 2 us.  Where 8 rows a workgroup are too many (d_model up to 1024: 128 workgroups), W_down
// goes by 4 rows x 256 bytes at four chunks, and a quarter of a product counts.  MFMAs are far from what bounds this.  x comes
// through LDS (direct loads of whole lines; from its rows into fragments 2 us more a token group of 8 at d_model 2048); H is exchanged in
// the order of the down product's fragments, 1 KB each.  The 8 wavefronts share K, and add up through LDS.
//
// The exchange.  H is stored and loaded with the device scope bit (sc1), past the L2s of the eight XCDs, which do not see each
// other's lines; a workgroup waits until its stores are complete and then raises its flag to the launch's number, and one wavefront looks at
// all flags at once.  There are 32 copies of the flags, each looked at by 8 workgroups: 256 that read the same 8 lines wait
// for each other (1.0 us a look; a layer of 512 x 1536, one token, with 1 / 8 copies 6.9 / 6.1 us, with 16 / 32 5.7 / 5.5).  The grid is the context's, not the
// call's, so every launch raises the same flags to the next number, which is never 0 (a claim nobody has made): nothing is reset, and a
// graph replays it.
//
// Workgroups wait for workgroups, so what a launch shares the chip with matters: a compute unit is held until the launch is resident as a
// whole.  Therefore two workgroups fit a compute unit (registers: 128, which takes recomputed indices, scalar offsets and, for the widest
// layers, fewer early loads; LDS: up to 80 KB, which bounds d_model times tokens; see FIT).  Two launches side by side are then resident
// together, a third gets in when one of them ends.  With one a compute unit, three launches at a time kept each other off the chip until
// somebody gave up: eight layers of 2048 x 8192, one token, us a step of each stream, two launches a layer / this, one a compute unit / this,
// two: 2 at a time 210 / 222 / 196, 4 streams 315 / 7760 / 266; beside a prefill of 4096 tokens 1064 / 1107 / 700 to 780, whose own call took
// 265 / 415 / 305 (257 alone).  1024 x 4096, 32 tokens, 4 streams 212 / 7860 / 192.
//
// Nobody waits for good, as other streams may fill the chip all the same: one that has looked `looks` times
// gives its rows up by writing the launch's number into its claim, looks at the flags once more, and unless all are there, or it cannot
// take the claim back, ends.  Whoever sees all flags does its own rows and then those of every claim it can take.  No row is left: the
// workgroup whose flag was complete last sees all of them; who gave up before that has its claim complete before it looked at the
// flags the last time, where that last flag was missing, so the claim is there when the last workgroup reads it.  (Each takes a claim back to
// 0 by compare and swap, so a share is done once.)  Workgroups begin their search for claims at different ones, and load them anew where
// another was faster.  us a round of 8 streams (seven decode steps of 2048 x 8192 and 1024 x 4096, 1 to 32 tokens, one of 512 x 1536, all at
// once; two launches a layer 990) by the number of looks, searches in one order / in different ones: 2000 3700 / 3380, 400 2300 / 1420, 200 1700 / 1190, 100 1310 /
// 1190, 50 - / 1300, 20 - / 2330; of five decode steps and three prefills on 8 streams (770) at 400 looks 1020 / 995, 200 985 / 935, 100 970 / 905.
// (Workgroups that give up one after another, over nine times as many looks: 1600 and 1080 at 50.)  On four streams two decode
// steps and two prefills take 358, four decode steps 345, where two launches a layer take 385 and 365.
//
// Layer forward, us, two launches of the decode kernel / this, 1, 8, 16, 24, 32 tokens, 16 or 24 layers in a graph: 512 x 1536 7.0 / 5.4, 7.3 / 5.6, 7.7 / 5.8,
// 8.3 / 6.3, 8.6 / 6.8; 1024 x 4096 9.4 / 8.0, 9.9 / 8.1, 11.3 / 8.7, 12.0 / 9.7, 12.3 / 10.6; 1536 x 5120 12.4 / 9.9, 13.4 / 9.8, 15.2 / 11.1,
// 16.4 / 12.3; 2048 x 8192 17.2 / 16.0, 17.3 / 15.9, 18.8 / 18.2.  What bounds it, from stamps of one workgroup a compute unit, 24 tokens
// at 1024 x 4096: first W_gate bytes 1.0 us after the start, all of them 2.7, H complete 3.7 (the last workgroup's 4.7), everybody through
// 5.6, H read 7.5 (196 KB a compute unit from L2), end 8.3; one token at 2048 x 8192: the weights, 12.4 of 14 us.  (Without W_down before the
// exchange 1536 x 5120 and above 0.5 to 0.7 us more; all of it before, 0.1 to 0.9.  H loaded without the scope bit: the same.)
#include <type_traits>

#include "stem_internal.h"

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;
typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef __amdgpu_buffer_rsrc_t rsrc_t;

namespace {

constexpr int WAVES = 8, THREADS = 64 * WAVES, MAX_WGS = 256;
constexpr uint32_t OOB = 0x80000000u;   // a buffer offset beyond any operand: reads as zero
constexpr int SC1 = 16;                 // cache policy bit of the buffer instructions: device scope
constexpr int REPLICAS = 32;            // of the flags
constexpr int FLIGHT = 8;               // fragments of H a wavefront has in flight at least

struct Args {
  const bf16_t *x, *Wg, *Wd, *E, *residual;
  const int32_t* ids;
  bf16_t *y, *H, *save_G, *save_H;      // H: the exchange's; the saved ones may be null
  uint32_t* sync;                       // 32 x 256 flags, 256 claims
  int32_t* bad_id;
  int T, d, F, E_rows, looks;
};

__device__ __forceinline__ float sigmoidf_fast(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }
__device__ __forceinline__ u32x2_t pack4(const float (&f)[4]) {
  bf16x4_t v;
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] = (__bf16)f[q];
  return __builtin_bit_cast(u32x2_t, v);
}
__device__ __forceinline__ void unpack4(u32x2_t v, float (&f)[4]) {
  f[0] = __uint_as_float(v[0] << 16); f[1] = __uint_as_float(v[0] & 0xffff0000u);
  f[2] = __uint_as_float(v[1] << 16); f[3] = __uint_as_float(v[1] & 0xffff0000u);
}
template <class P>
__device__ __forceinline__ rsrc_t rsrc(P* p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(static_cast<const void*>(p)), 0, bytes, 0x00020000);
}
template <int AUX>
__device__ __forceinline__ bf16x8_t load16(rsrc_t r, uint32_t off, int scalar_off = 0) {
  return __builtin_bit_cast(bf16x8_t, __builtin_amdgcn_raw_buffer_load_b128(r, off, scalar_off, AUX));
}
__device__ __forceinline__ void keep_order() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
// v for uses from here on: what they compute from it is not kept in registers from earlier ones
__device__ __forceinline__ int afresh(int v) {
  asm volatile("" : "+v"(v));
  return v;
}
__device__ __forceinline__ f32x4_t mfma(bf16x8_t w, bf16x8_t t, f32x4_t acc) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, t, acc, 0, 0, 0);
}

__device__ __forceinline__ float add_neighbour(float v) {   // lane ^ 1
  return v + __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0xb1, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ void add_dpp(f32x4_t& s) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float v = s[q];
    s[q] = v + __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), CTRL, 0xf, 0xf, true));
  }
}
// The sum of the wavefronts' partial sums, REGION floats apart, by S = 1, 2, 4 or 8 neighbouring lanes, the `s`-th of which this is; each
// gets it.
template <int S, int REGION>
__device__ __forceinline__ f32x4_t sum_partials(const float* from, int s) {
  constexpr int N = WAVES / S;
  f32x4_t v[N];
#pragma unroll
  for (int q = 0; q < N; ++q) v[q] = *reinterpret_cast<const f32x4_t*>(from + (s * N + q) * REGION);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int n = 1; n < N; n *= 2)
#pragma unroll
    for (int q = 0; q + n < N; q += 2 * n) v[q] += v[q + n];
  if (S > 1) add_dpp<0xb1>(v[0]);    // quad_perm 1 0 3 2
  if (S > 2) add_dpp<0x4e>(v[0]);    // quad_perm 2 3 0 1
  if (S > 4) add_dpp<0x141>(v[0]);   // row_half_mirror
  return v[0];
}

// RG x 8 columns of H a workgroup (d_ff up to RG * 2048), KG lines of 64 k a wavefront (d_model up to KG * 512), up to 8 TQ tokens,
// RD = 8 or 4 rows of W_down a workgroup.  LDS is 8 KB * KG * TQ: two workgroups fit a compute unit up to 9 of these.
constexpr int FIT = 9;
template <int RG, int KG, int TQ, int RD>
__global__ __launch_bounds__(THREADS, 4) void ffn_decode_kernel(Args p) {
  constexpr int TM = 8 * TQ;
  // Cache policy of the weights.  The last level holds 256 MB: weights of a stack that fits are best kept there, others best read past it
  // (policy 2).  A call doesn't know the stack: of layers up to 8.4 MB (RG * KG up to 2) twenty or thirty fit, of larger ones they don't.
  // us a layer, kept / past it, one token: 512 x 1536 (3.1 MB) 8 layers 5.6 / 5.7, 24 5.4 / 5.6, 48 5.3 / 5.5; 1024 x 4096 (16.8 MB) 8 layers 7.8 / 8.3,
  // 16 7.8 / 8.0, 24 8.2 / 8.0, 48 8.1 / 7.9; 1536 x 5120 8 layers 9.7 / 10.2, 16 10.3 / 9.9, 48 9.9 / 9.5; 2048 x 8192 4 layers 17.0 / 16.5, 8 17.6 /
  // 16.1, 16 17.2 / 15.9, 48 16.6 / 15.7.
  constexpr int KEEP = RG * KG <= 2 ? 0 : 2;
  constexpr int LD = RD == 8 ? 1 : 2;                                        // lines of 64 k in a piece of W_down
  constexpr int KD = 4 * RG / LD;                                            // pieces a wavefront
  constexpr int EARLY = RG * KG >= 12 && TQ >= 2 ? 2 : KD / 2;               // requested at the start (where registers are short: few)
  constexpr int GP = 8 * RG + 4, DP = RD == 8 ? 12 : 4;                      // floats between two tokens' sums in LDS
  // LDS, a region for each wavefront: its part of x, then its partial sums
  constexpr int XB = KG * TQ * 1024, GB = TM * GP * 4, DB = TM * DP * 4, REGION = XB > GB ? (XB > DB ? XB : DB) : (GB > DB ? GB : DB);
  __shared__ __attribute__((aligned(16))) char smem[WAVES * REGION + 16];   // (one variable: see the wait for x)
  float* const red = reinterpret_cast<float*>(smem);
  int* const next_share = reinterpret_cast<int*>(smem + WAVES * REGION);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // a fragment's lane: row or token o of 8, and of a line's 8 chunks of 8 k the c-th of the g-th two
  const int c = lane & 1, o = lane >> 1 & 7, g = lane >> 4;
  const int b = blockIdx.x, wgs = gridDim.x;
  const bool gate = b * 8 * RG < p.F, down = b * RD < p.d;
  const rsrc_t rflags = rsrc(p.sync, REPLICAS * MAX_WGS * 4), rclaims = rsrc(p.sync + REPLICAS * MAX_WGS, MAX_WGS * 4);
  const rsrc_t rH = rsrc(p.H, (p.F + 64 * LD - 1) / (64 * LD) * LD * p.T * 128);

  const uint32_t epoch = stem_launch_after(__builtin_amdgcn_raw_buffer_load_b32(rflags, b * 4, 0, SC1));

  // ---- all loads: ids, W_gate and x, the table rows, W_down, the residual.  None is conditional, or the compiler waits for all of those it
  // cannot count: what a workgroup has no part in is read out of range or for nothing.
  // H by 4 columns of a token, HS lanes each: thread -> (token, chunk of 8 columns, half of the chunk, lane)
  constexpr int HQ = TM * RG * 2, HS = THREADS / HQ < 4 ? (THREADS / HQ < 2 ? 1 : 2) : 4;
  static_assert(HQ <= THREADS, "a thread for each");
  const int h_s = tid % HS, h_half = tid / HS & 1, h_chunk = tid / (2 * HS) % RG, h_tok = tid / (2 * HS * RG);
  const int h_col_raw = (b * RG + h_chunk) * 8 + h_half * 4;
  const bool has_h = h_col_raw < p.F && h_tok < p.T;
  const int id_raw = p.ids[h_tok < p.T ? h_tok : p.T - 1];
  bf16x8_t w[KG][RG], x[KG][TQ];
  char* const region = smem + wave * REGION;
  {
    // x straight to LDS by 8 tokens x 128 bytes, eight lanes a line: 16-byte chunk c of token o's line lies at chunk c ^ (o & 6)
    const rsrc_t rw = rsrc(p.Wg, p.F * p.d * 2), rx = rsrc(p.x, p.T * p.d * 2);
#pragma unroll
    for (int i = 0; i < KG; ++i)
#pragma unroll
      for (int t = 0; t < TQ; ++t) {
        const int kl = wave + WAVES * i, tok = t * 8 + (lane >> 3);
        const uint32_t off = (uint32_t)(tok * p.d + ((lane & 7) ^ (lane >> 3 & 6)) * 8) * 2;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_ptr_t)(region + (i * TQ + t) * 1024), 16,
                                                 off | (tok < p.T && kl * 64 < p.d && gate ? 0 : OOB), kl * 128, 0, 0);
      }
    keep_order();
    const uint32_t ow = (uint32_t)((b * 8 * RG + o) * p.d + (2 * g + c) * 8) * 2;
#pragma unroll
    for (int i = 0; i < KG; ++i) {
      const int kl = wave + WAVES * i;
#pragma unroll
      for (int r = 0; r < RG; ++r) w[i][r] = load16<KEEP>(rw, (ow + (uint32_t)(r * 8 * p.d * 2 + kl * 128)) | (kl * 64 < p.d && gate ? 0 : OOB));
    }
  }
  keep_order();
  const bool bad = has_h && (unsigned)id_raw >= (unsigned)p.E_rows;   // reported below, clamped so no access leaves the table
  const int id = id_raw < 0 ? 0 : id_raw < p.E_rows ? id_raw : p.E_rows - 1;
  const int h_col = h_col_raw < p.F ? h_col_raw : 0;
  const u32x2_t ev = *reinterpret_cast<const u32x2_t*>(p.E + (size_t)id * p.F + h_col);
  keep_order();
  const rsrc_t rwd = rsrc(p.Wd, p.d * p.F * 2);
  // y by 4 rows of a token, YS lanes each: thread t's
  constexpr int YQ = TM * RD / 4, YS = THREADS / YQ < 8 ? THREADS / YQ < 4 ? 2 : 4 : 8;
  auto y_row = [](int t) { return RD == 8 ? (t / YS & 1) * 4 : 0; };
  auto y_tok = [](int t) { return t / (YS * (RD / 4)); };
  const bf16_t* const residual = p.residual ? p.residual : p.x;
  bf16x8_t wd[KD];
  u32x2_t rv;
  auto load_share = [&](int share, bool mine, int from, int to) __attribute__((always_inline)) {
    const int t = afresh(tid), lane = t & 63;
    const int row = RD == 8 ? lane >> 1 & 7 : lane >> 2 & 3, chunk = RD == 8 ? 2 * (lane >> 4) + (lane & 1) : 4 * (lane >> 4) + (lane & 3);
    const uint32_t at = (uint32_t)((share * RD + row) * p.F + chunk * 8) * 2 | (mine ? 0 : OOB);
#pragma unroll
    for (int i = 0; i < KD; ++i) {
      const int k = (wave + WAVES * i) * 64 * LD;
      if (i >= from && i < to)                                // (d_ff is whole lines: a piece of one is in range or not)
        wd[i] = LD == 1 ? load16<KEEP>(rwd, k < p.F ? at : OOB, k * 2) : load16<KEEP>(rwd, (at + k * 2) | (k + chunk * 8 < p.F ? 0 : OOB));
    }
    if (to == KD)
      rv = *reinterpret_cast<const u32x2_t*>(residual + (size_t)(y_tok(t) < p.T ? y_tok(t) : p.T - 1) * p.d + (mine ? share : 0) * RD + y_row(t));
  };
  if (EARLY) load_share(b, down, 0, EARLY);
  keep_order();

  // ---- gate product
  // x is there when no more than the loads behind it are outstanding.  (The table rows' is not counted: whatever the compiler makes of
  // it, the wait is then long enough.)
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(KG * RG + EARLY) : "memory");
  if (gate) {
#pragma unroll
    for (int i = 0; i < KG; ++i)
#pragma unroll
      for (int t = 0; t < TQ; ++t) x[i][t] = *reinterpret_cast<const bf16x8_t*>(region + (i * TQ + t) * 1024 + o * 128 + (((2 * g + c) ^ (o & 6)) << 4));
    f32x4_t acc[RG][TQ];
#pragma unroll
    for (int r = 0; r < RG; ++r)
#pragma unroll
      for (int t = 0; t < TQ; ++t) acc[r][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < KG; ++i)
#pragma unroll
      for (int r = 0; r < RG; ++r)
#pragma unroll
        for (int t = 0; t < TQ; ++t) acc[r][t] = mfma(w[i][r], x[i][t], acc[r][t]);
    // of a product a lane holds rows 4 g .. 4 g + 3, weight rows 2 g and 2 g + 1 at either chunk, by token o at chunk c
#pragma unroll
    for (int r = 0; r < RG; ++r)
#pragma unroll
      for (int t = 0; t < TQ; ++t) {
        const float lo = add_neighbour(c ? acc[r][t][1] : acc[r][t][0]), hi = add_neighbour(c ? acc[r][t][3] : acc[r][t][2]);
        *reinterpret_cast<float*>(region + ((t * 8 + o) * GP + r * 8 + 2 * g + c) * 4) = c ? hi : lo;
      }
  }
  __syncthreads();
  if (has_h) {
    const f32x4_t s = sum_partials<HS, REGION / 4>(red + h_tok * GP + h_chunk * 8 + h_half * 4, h_s);
    float e[4], v[4];
    unpack4(ev, e);
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = s[q] * sigmoidf_fast(s[q]) * e[q];
    // by the down product's fragments, of these by 8 tokens, and then in the order of a fragment's lanes
    const int chunk = h_col >> 3, octet = h_tok & ~7, in = p.T - octet < 8 ? p.T - octet : 8;
    const int frag = RD == 8 ? chunk >> 3 : (chunk >> 4) * 2 + (chunk >> 1 & 1), hg = RD == 8 ? chunk >> 1 & 3 : chunk >> 2 & 3;
    if (h_s == 0)
      __builtin_amdgcn_raw_buffer_store_b64(pack4(v), rH, (frag * p.T + octet) * 128 + ((hg * in + (h_tok & 7)) * 2 + (chunk & 1)) * 16 + h_half * 8, 0, SC1);
    if (h_s == 0 && p.save_G) *reinterpret_cast<u32x2_t*>(p.save_G + (size_t)h_tok * p.F + h_col) = pack4({s[0], s[1], s[2], s[3]});
    if (h_s == 0 && p.save_H) *reinterpret_cast<u32x2_t*>(p.save_H + (size_t)h_tok * p.F + h_col) = pack4(v);
    if (bad) *p.bad_id = 1;
  }
  keep_order();
  load_share(b, down, EARLY, KD);
  keep_order();
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(KD - EARLY + 1) : "memory");   // what is stored is complete for the device
  __syncthreads();

  // ---- the exchange
  u32x4_t claims = {};
  constexpr int LOOKS = WAVES - 1;   // the wavefront that looks: the first ones have H to store and wait for (0.1 to 0.3 us)
  if (wave == LOOKS) {
    if (lane < REPLICAS) __builtin_amdgcn_raw_buffer_store_b32(epoch, rflags, (lane * MAX_WGS + b) * 4, 0, SC1);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // complete before it looks at the others'
    auto all_there = [&]() __attribute__((always_inline)) {
      asm volatile("" ::: "memory");                     // every look is a load
      const u32x4_t f = __builtin_amdgcn_raw_buffer_load_b128(rflags, (b / 8 % REPLICAS * MAX_WGS + lane * 4) * 4, 0, SC1);
      const int n = wgs - lane * 4;                      // flags of this lane
      return __ballot((n > 0 && f[0] != epoch) || (n > 1 && f[1] != epoch) || (n > 2 && f[2] != epoch) || (n > 3 && f[3] != epoch)) == 0;
    };
    bool there = all_there();
    for (int n = down ? p.looks : 0; !there && n > 0; --n) there = all_there();
    bool mine = there && down;
    if (!there && down) {            // give the share up
      uint32_t* const claim = p.sync + REPLICAS * MAX_WGS + b;
      if (lane == 0) __hip_atomic_store(claim, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      there = all_there();
      if (there) {                   // or take it back
        uint32_t was = epoch;
        bool got = false;
        if (lane == 0) got = __hip_atomic_compare_exchange_strong(claim, &was, 0u, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        mine = __ballot(got) != 0;
      }
    }
    // (a wavefront's lane l holds claims 4 l .. 4 l + 3; requested here, looked at when the own share is done)
    asm volatile("" ::: "memory");
    if (there) claims = __builtin_amdgcn_raw_buffer_load_b128(rclaims, lane * 16, 0, SC1);
    if (lane == 0) *next_share = mine ? b : there ? -1 : -2;   // -1: only other workgroups' shares, -2: none
  }
  __syncthreads();
  int share = *next_share;
  if (share == -2) return;

  // ---- down product: the own share, then those given up
  for (;;) {
    if (share >= 0) {
      constexpr int FD = LD * TQ;                                   // fragments, and accumulators, of a piece
      constexpr int BATCH = FLIGHT / FD > KD ? KD : FLIGHT / FD > 0 ? FLIGHT / FD : 1;    // pieces whose fragments are in flight together
      const int l = afresh(lane), c = l & 1, o = l >> 1 & 7, g = l >> 4;
      f32x4_t acc[FD];
#pragma unroll
      for (int f = 0; f < FD; ++f) acc[f] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      uint32_t oh[TQ];
#pragma unroll
      for (int t = 0; t < TQ; ++t) {
        const int in = p.T - t * 8 < 8 ? p.T - t * 8 : 8;           // (as they were stored)
        oh[t] = (uint32_t)(t * 1024 + ((g * in + o) * 2 + c) * 16) | (o < in ? 0 : OOB);
      }
#pragma unroll
      for (int i0 = 0; i0 < KD; i0 += BATCH) {
        bf16x8_t v[BATCH][FD];
#pragma unroll
        for (int i = 0; i < BATCH; ++i)
#pragma unroll
          for (int f = 0; f < FD; ++f)                              // beyond d_ff: reads as zero
            if (i0 + i < KD) {
              const int piece = wave + WAVES * (i0 + i), k = piece * 64 * LD + (4 * g + f / TQ * 2 + c) * 8;
              v[i][f] = LD == 1 ? load16<SC1>(rH, piece * 64 < p.F ? oh[f] : OOB, piece * p.T * 128)
                                : load16<SC1>(rH, (oh[f % TQ] + (piece * LD + f / TQ) * p.T * 128) | (k < p.F ? 0 : OOB));
            }
        keep_order();
#pragma unroll
        for (int i = 0; i < BATCH; ++i)
#pragma unroll
          for (int f = 0; f < FD; ++f)
            if (i0 + i < KD) acc[f] = mfma(wd[i0 + i], v[i][f], acc[f]);
        keep_order();
      }
      // as above; or of a piece of 4 rows a lane holds row g at four chunks, by two fragments of two chunks
#pragma unroll
      for (int t = 0; t < TQ; ++t) {
        const f32x4_t a0 = acc[t], a1 = acc[(TQ + t) % FD];
        if (RD == 8) {
          const float lo = add_neighbour(c ? a0[1] : a0[0]), hi = add_neighbour(c ? a0[3] : a0[2]);
          *reinterpret_cast<float*>(region + ((t * 8 + o) * DP + 2 * g + c) * 4) = c ? hi : lo;
        } else {
          const float sum = add_neighbour((c ? a0[1] : a0[0]) + (c ? a1[3] : a1[2]));
          if (c == 0) *reinterpret_cast<float*>(region + ((t * 8 + o) * DP + g) * 4) = sum;
        }
      }
      __syncthreads();
      const int t = afresh(tid), tok = y_tok(t), row = y_row(t), y_s = t % YS;
      if (tok < p.T) {
        const f32x4_t s = sum_partials<YS, REGION / 4>(red + tok * DP + row, y_s);
        float out[4] = {s[0], s[1], s[2], s[3]};
        if (p.residual) {   // the layer's output joins the residual stream: added in fp32, rounded once
          float r[4];
          unpack4(rv, r);
#pragma unroll
          for (int q = 0; q < 4; ++q) out[q] += r[q];
        }
        if (y_s == 0) *reinterpret_cast<u32x2_t*>(p.y + (size_t)tok * p.d + share * RD + row) = pack4(out);
      }
    } else {
      __syncthreads();   // all have read next_share
    }
    // a share that was given up, if there is one: the claims that were there, one after another
    if (wave == LOOKS) {
      int found = -1;
      const int turn = b * 37 >> 2 & 63;                   // where this workgroup begins to look
      for (;;) {
        uint64_t any = __ballot(claims[0] == epoch || claims[1] == epoch || claims[2] == epoch || claims[3] == epoch);
        if (!any) break;
        any = any >> turn | any << (63 - turn) << 1;
        const int from = (__builtin_ctzll(any) + turn) & 63;
        bool got = false;
        int which = 0;
        if (lane == from) {
          which = claims[0] == epoch ? 0 : claims[1] == epoch ? 1 : claims[2] == epoch ? 2 : 3;
          uint32_t was = epoch;
          got = __hip_atomic_compare_exchange_strong(p.sync + REPLICAS * MAX_WGS + lane * 4 + which, &was, 0u, __ATOMIC_RELAXED,
                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          claims[which] = 0;
        }
        which = __builtin_amdgcn_readlane(which, from);
        if (__ballot(got)) { found = from * 4 + which; break; }
        asm volatile("" ::: "memory");                     // another workgroup was faster: what is there now
        claims = __builtin_amdgcn_raw_buffer_load_b128(rclaims, lane * 16, 0, SC1);
      }
      if (lane == 0) *next_share = found;
    }
    __syncthreads();
    share = *next_share;
    if (share < 0) return;
    load_share(share, true, 0, KD);
  }
}

template <int RG, int KG, int RD>
void launch(const Args& p, int wgs, hipStream_t s) {
  auto* kernel = p.T <= 8 ? ffn_decode_kernel<RG, KG, 1, RD> : ffn_decode_kernel<RG, KG, 2, RD>;
  if constexpr (KG * 3 <= FIT)
    if (p.T > 16) kernel = ffn_decode_kernel<RG, KG, 3, RD>;
  if constexpr (KG * 4 <= FIT)
    if (p.T > 24) kernel = ffn_decode_kernel<RG, KG, 4, RD>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)wgs), dim3(THREADS), 0, s, p);
}

}  // namespace

// Up to 32 tokens: every workgroup reads all tokens' H, and a lane's sums of more don't fit its registers.  And while two workgroups fit a
// compute unit: up to 32 tokens of d_model up to 1024, 24 up to 1536, 16 up to 2048.  (One a compute unit, by itself, two launches /
// this: 1536 x 5120, 32 tokens 17.3 / 13.7; 2048 x 8192, 24 and 32 20.2 / 18.9, 21.5 / 20.9; 48 tokens of 512 x 2048 10.5 / 7.9, of
// 1024 x 4096 13.2 / 12.4.  Three of them at a time take ten times as long as two launches a layer do.)  Wider layers do not fit a workgroup's registers.
int stem_route_one_launch(int d, int F, int64_t T) {
  return T >= 1 && T <= 32 && d % 64 == 0 && F % 64 == 0 && d <= 2048 && F <= 8192 && (d + 511) / 512 * ((T + 7) / 8) <= FIT;
}

// Two launches store G and H before W_down and the residual are read and y is stored; here other workgroups do the one while some do the
// other.
int stem_route_one_launch_apart(int d, int F, int64_t T, const void* G, const void* H, const void* W_down, const void* residual,
                                const void* y) {
  const struct { const void* at; size_t n; } out[] = {{G, (size_t)T * F * 2}, {H, (size_t)T * F * 2}},
      other[] = {{W_down, (size_t)F * d * 2}, {residual, (size_t)T * d * 2}, {y, (size_t)T * d * 2}};
  for (const auto& a : out)
    for (const auto& b : other) {
      const uintptr_t x = reinterpret_cast<uintptr_t>(a.at), z = reinterpret_cast<uintptr_t>(b.at);
      if (x && z && x < z + b.n && z < x + a.n) return 0;
    }
  return 1;
}

uint32_t stem_next_launch(uint32_t last) { return stem_launch_after(last); }

int stem_exchange_launch(stem_ctx* c, uint32_t last) {
  hipError_t e = hipDeviceSynchronize();
  if (e == hipSuccess) e = hipMemsetD32(reinterpret_cast<hipDeviceptr_t>(c->sync), (int)last, REPLICAS * MAX_WGS);
  return e != hipSuccess ? e : hipDeviceSynchronize();
}

hipError_t stem_ffn_decode_bf16(stem_ctx* ctx, const StemDecodeArgs& a, hipStream_t s) {
  if (!stem_route_one_launch(a.d, a.F, a.T)) return hipErrorInvalidValue;
  Args p;
  p.x = a.x; p.Wg = a.Wg; p.Wd = a.Wd; p.E = a.E; p.residual = a.residual; p.ids = a.ids; p.y = a.y; p.save_G = a.save_G; p.save_H = a.save_H;
  p.H = reinterpret_cast<bf16_t*>(ctx->splitk_ws); p.sync = ctx->sync; p.bad_id = ctx->flag;
  p.T = a.T; p.d = a.d; p.F = a.F; p.E_rows = a.E_rows; p.looks = ctx->looks;
  const int rg = (a.F + 2047) / 2048, rd = a.d <= 1024 ? 4 : 8;
  const int gates = (a.F + 8 * rg - 1) / (8 * rg), downs = a.d / rd, wgs = gates > downs ? gates : downs;
  ProfScope ps(ctx, K_FFN_DECODE, s);
  const auto by_rg = [&](auto kg, auto rd_c) {
    constexpr int KG = decltype(kg)::value, RD = decltype(rd_c)::value;
    rg == 1 ? launch<1, KG, RD>(p, wgs, s) : rg == 2 ? launch<2, KG, RD>(p, wgs, s) : rg == 3 ? launch<3, KG, RD>(p, wgs, s) : launch<4, KG, RD>(p, wgs, s);
  };
  std::integral_constant<int, 4> four;
  std::integral_constant<int, 8> eight;
  if (a.d <= 512) by_rg(std::integral_constant<int, 1>(), four);
  else if (a.d <= 1024) by_rg(std::integral_constant<int, 2>(), four);
  else if (a.d <= 1536) by_rg(std::integral_constant<int, 3>(), eight);
  else by_rg(std::integral_constant<int, 4>(), eight);
  return hipGetLastError();
}
