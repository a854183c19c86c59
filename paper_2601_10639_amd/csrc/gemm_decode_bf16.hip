// bf16 MFMA products of a decode step (one token to a few hundred), gfx950.
//
// C[m,n] = sum_k A[m,k] * B[n,k], both operands K-contiguous, B the weights.  At these sizes a launch takes 5 to 20 us
// and is bound by how early and how densely the operand bytes are requested: the 33 MB of one weight matrix
// (d_model 2048, d_ff 8192) are 5.5 us of HBM time, and every workgroup reads its token rows from L2 besides.
//
// The tile is TM tokens x TN weight rows, and the W wavefronts of a workgroup share it by splitting K: wavefront w
// takes every W-th K tile (64 wide) of the whole tile.  So no operand byte is loaded twice by a workgroup, nothing
// passes between wavefronts until the end, and the main loop has no barrier: each wavefront fills a ring of D K tiles
// of its own in LDS by direct loads of whole 128-byte lines (both operands; 100 to 130 KB in flight per CU) and waits
// for its oldest by count.  (Weights or both operands loaded straight into MFMA fragments, 16 rows x 64 bytes per
// instruction, took 1 to 3 us longer per launch from 16 tokens on: half lines.  Two wavefronts per row half with one
// ring for the workgroup and a barrier per K tile, the few-row kernel's scheme, 15.6 us instead of 8.1 at one token.)
// (Requests past the last K tile that go to an empty buffer would keep that count the same throughout, but cost 0.7 us
// of a launch: an empty load still writes LDS.)
//
// At the end the W partial tiles are added through LDS in wavefront order, and all threads run the epilogue on 4
// consecutive n each.
//
// Split K (the down product: few output tiles, long K).  Each slice writes its fp32 tile to the workspace and takes a
// ticket of its tile; the workgroup that takes the last one adds the slices in slice order, whichever it is.  Nobody
// waits for anybody.  The slices of a tile run on different XCDs, whose L2s do not see each other's lines; the partial
// tiles therefore bypass them: stores and loads carry the device scope bit (sc1), a store is complete for the device
// when it leaves vmcnt, and every wavefront waits for that before the workgroup's ticket is taken.  That orders the
// exchange without a device-scope fence, which would write back or drop the whole L2 under the weight streams of the
// other workgroups (20 -> 41 us when this was tried with fences).  2048 x 8192 down product, 16 tokens: 12.5 us
// unsplit, 9.9 in two slices; against 10.6 + 3.9 for a split product and a kernel that sums.
#include "stem_internal.h"

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef __amdgpu_buffer_rsrc_t rsrc_t;

namespace {

constexpr int BK = 64;
constexpr uint32_t OOB = 0x80000000u;   // a buffer offset beyond any operand: reads as zero
constexpr int SC1 = 16;                 // cache policy bit of the buffer instructions: device scope
constexpr int MAX_SLICES = 8;

__device__ __forceinline__ float sigmoidf_fast(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }
__device__ __forceinline__ uint2 pack4(const float (&f)[4]) {
  bf16x4_t v;
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] = (__bf16)f[q];
  return __builtin_bit_cast(uint2, v);
}
// 16-byte chunk c of row r of a K tile (128 bytes a row) sits at chunk slot c ^ swz(r): the 16 rows of a fragment read
// then touch all banks once
__device__ __forceinline__ int swz(int r) { return (r >> 1) & 7; }
__device__ __forceinline__ void lds_dma_16(rsrc_t rs, char* lds_dst, uint32_t off, int soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)lds_dst, 16, off, soff, 0, 0);
}

// Waits until at most min(younger, MOST) K tiles of LOADS loads each are outstanding; the count is an immediate.  It
// counts the K tiles alone, each of them exactly LOADS instructions: whatever else a wavefront has in flight, and however
// many instructions the compiler makes of it, only makes the wait longer.  (Counting the gate product's table-row loads in
// as well is 0.1 us shorter where a wavefront has one K tile, and reads a K tile too early if they become fewer.)
template <int LOADS, int MOST>
__device__ __forceinline__ void wait_all_but(int younger) {
  if (MOST == 0 || younger >= MOST) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(MOST * LOADS) : "memory");
  else wait_all_but<LOADS, (MOST > 0 ? MOST - 1 : 0)>(younger);
}

// FA x 16 tokens, FB x 16 weight rows, W wavefronts with D K tiles in flight each
template <int FA_, int FB_, int W_, int D_>
struct Shape {
  static constexpr bool PAIR = false;
  static constexpr int FA = FA_, FB = FB_, W = W_, D = D_, RM = 16 * FA, RN = 16 * FB;   // rows of a K tile in LDS
  static constexpr int TM = RM, TN = RN, KW = BK;           // the output tile, K of a K tile
  static constexpr int SLOT = (RM + RN) * BK * 2;           // one K tile of both operands
  static constexpr int PITCH = RN + 4;                      // floats per row of a partial tile in LDS
  static constexpr int RING = W * D * SLOT, RED = W * RM * PITCH * 4;
  static constexpr int LDS_BYTES = RING > RED ? RING : RED;
};
// 8 tokens x 8 weight rows, K tiles 128 wide: rows 0-7 of a fragment are the 8 rows at the first half of the K tile, rows
// 8-15 the same rows at the second, and of the 16 x 16 products the two diagonal 8 x 8 blocks are the sums of the halves.
template <int W_, int D_>
struct PairShape : Shape<1, 1, W_, D_> {
  static constexpr bool PAIR = true;
  static constexpr int TM = 8, TN = 8, KW = 2 * BK;
};

template <class S, int EPI>
__global__ __launch_bounds__(64 * S::W) void gemm_decode_kernel(GemmArgs p) {
  constexpr int FA = S::FA, FB = S::FB, W = S::W, D = S::D, TM = S::TM, TN = S::TN, RM = S::RM, KW = S::KW;
  constexpr int QUADS = TM * TN / 4, QT = (QUADS + 64 * W - 1) / (64 * W);   // quads of 4 columns; per thread
  constexpr int LOADS = 2 * (FA + FB);                                       // per wavefront and K tile
  __shared__ __attribute__((aligned(16))) char smem[S::LDS_BYTES];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // Workgroup -> (token tile, weight tile, K slice): each XCD gets a contiguous run of the linear order, in which the
  // token tiles of one weight tile are neighbours, so the weight rows they share come from HBM once.  (The quotients
  // are below 2^20: the float reciprocals are exact here.)
  int tm, tn, z;
  {
    const int nb = gridDim.x, b = blockIdx.x;
    const int q = nb >> 3, r = nb & 7;
    const int xcd = b & 7, idx = b >> 3;
    const int L = xcd * q + (xcd < r ? xcd : r) + idx;
    const int per_z = p.mt * p.nt;
    z = (int)(((float)L + 0.5f) * p.inv_per_z);
    const int in = L - z * per_z;
    tn = (int)(((float)in + 0.5f) * p.inv_mt);
    tm = in - tn * p.mt;
  }
  const int m0 = tm * TM, n0 = tn * TN;
  const int nk_all = (p.K + KW - 1) / KW, per = (nk_all + p.ksplit - 1) / p.ksplit, kt0 = z * per;
  const int nk = nk_all - kt0 < per ? nk_all - kt0 : per;      // at least 1

  // The gate epilogue multiplies by a gathered table row: its token ids are requested first of all, the row pieces
  // right behind the first K tiles, so that both pass under the main loop.
  int ids_q[QT];
  uint2 ev[QT];
  bool bad = false;
  if (EPI == EPI_GATE) {
#pragma unroll
    for (int q = 0; q < QT; ++q) {
      const int m = m0 + (q * 64 * W + tid) / (TN / 4);
      ids_q[q] = p.ids[m < p.M ? m : p.M - 1];
    }
  }

  // loads of a K tile: 8 rows x 128 bytes each, token rows first; lane -> row (lane >> 3), the chunk of its slot
  const rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p.A), 0, p.M * p.lda * 2, 0x00020000);
  const rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p.B), 0, p.N * p.ldb * 2, 0x00020000);
  uint32_t off[LOADS];
#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    const bool isA = i < 2 * FA;
    const int row = (isA ? i : i - 2 * FA) * 8 + (lane >> 3), g = (isA ? m0 : n0) + (S::PAIR ? row & 7 : row);
    const int k = ((lane & 7) ^ swz(row)) * 8 + (S::PAIR ? (row >> 3) * BK : 0);
    off[i] = g < (isA ? p.M : p.N) ? (uint32_t)((g * (isA ? p.lda : p.ldb) + k) * 2) : OOB;
  }
  // The walk over the K tiles starts at a place that differs from one weight tile to the next and wraps around:
  // operand rows are 2 to 16 KB apart, so their lines at one k sit in the same few memory channels.
  int kpos = (int)(((long)tn * nk) / p.nt) + wave;
  if (kpos >= nk) kpos -= nk;
  const int nw = nk > wave ? (nk - wave + W - 1) / W : 0;      // this wavefront's K tiles
  char* const ring = smem + wave * (D * S::SLOT);
  auto request = [&](int slot) __attribute__((always_inline)) {
    const int so = (kt0 + kpos) * (KW * 2);
    char* const dst = ring + slot * S::SLOT;
    if (S::PAIR) {   // the second half of the last K tile may lie beyond K: read as zero
      const bool whole = so + KW * 2 <= p.K * 2;
      const rsrc_t ra2 = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p.A), 0, whole ? p.M * p.lda * 2 : 0, 0x00020000);
      const rsrc_t rb2 = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p.B), 0, whole ? p.N * p.ldb * 2 : 0, 0x00020000);
      lds_dma_16(ra, dst, off[0], so);
      lds_dma_16(ra2, dst + 1024, off[1], so);
      lds_dma_16(rb, dst + 2048, off[2], so);
      lds_dma_16(rb2, dst + 3072, off[3], so);
    } else {
#pragma unroll
      for (int i = 0; i < LOADS; ++i) lds_dma_16(i < 2 * FA ? ra : rb, dst + i * 1024, off[i], so);
    }
    kpos += W;
    if (kpos >= nk) kpos -= nk;
  };

  // fragments: lane -> row (lane & 15) of 16, chunks (lane >> 4) and 4 + (lane >> 4) of its 128 bytes
  const int fr = lane & 15, fg = lane >> 4;
  const char* const frag = ring + fr * 128;
  const int c0 = ((fg ^ swz(fr)) & 7) << 4, c1 = (((4 + fg) ^ swz(fr)) & 7) << 4;
  f32x4_t acc[FA][FB];
#pragma unroll
  for (int a = 0; a < FA; ++a)
#pragma unroll
    for (int b = 0; b < FB; ++b) acc[a][b] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // The row pieces are younger than the first D K tiles and older than the rest; the barriers keep them in this place.
  auto load_rows = [&]() __attribute__((always_inline)) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < QT; ++q) {
      int id = ids_q[q];
      bad |= (unsigned)id >= (unsigned)p.E_rows;   // reported to the host below, clamped so no access leaves the table
      id = id < 0 ? 0 : id < p.E_rows ? id : p.E_rows - 1;
      const int n = n0 + ((q * 64 * W + tid) % (TN / 4)) * 4;
      ev[q] = *reinterpret_cast<const uint2*>(p.E + (size_t)id * p.N + (n < p.N ? n : 0));
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  // the usual case apart: behind conditional requests the compiler waits for all of them before it uses the ids
  if (nw >= D) {
#pragma unroll
    for (int d = 0; d < D; ++d) request(d);
    if (EPI == EPI_GATE) load_rows();
  } else {
#pragma unroll
    for (int d = 0; d < D - 1; ++d)
      if (d < nw) request(d);
    if (EPI == EPI_GATE) load_rows();
  }
  // lines past the end are empty loads, lines that a small grid does not come to are left out
  constexpr bool TOUCH = EPI == EPI_GATE && FA == 4;   // stem_touch_bytes: not for a few tokens
  uint32_t touched[4] = {};
  if (TOUCH && p.next_bytes) {
    const rsrc_t rn = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p.next), 0, p.next_bytes, 0x00020000);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      touched[i] = __builtin_amdgcn_raw_buffer_load_b32(rn, ((i * gridDim.x + blockIdx.x) * blockDim.x + tid) * 128, 0, 0);
  }
  int slot = 0;
  for (int i = 0; i < nw; ++i) {
    wait_all_but<LOADS, D - 1>(nw - 1 - i);
    const char* const f = frag + slot * S::SLOT;
    bf16x8_t xa[2][FA], xb[2][FB];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int b = 0; b < FB; ++b) xb[h][b] = *reinterpret_cast<const bf16x8_t*>(f + RM * 128 + b * 2048 + (h ? c1 : c0));
#pragma unroll
      for (int a = 0; a < FA; ++a) xa[h][a] = *reinterpret_cast<const bf16x8_t*>(f + a * 2048 + (h ? c1 : c0));
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the slot has been read: it may be filled again
    __builtin_amdgcn_sched_barrier(0);
    if (i + D < nw) request(slot);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int a = 0; a < FA; ++a)
#pragma unroll
        for (int b = 0; b < FB; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xb[h][b], xa[h][a], acc[a][b], 0, 0, 0);
    slot = slot + 1 == D ? 0 : slot + 1;
  }
  asm volatile("s_barrier" ::: "memory");            // nothing lands in LDS any more: every K tile has been waited for

  if (TOUCH) {   // the touching loads end here
#pragma unroll
    for (int i = 0; i < 4; ++i) asm volatile("" ::"v"(touched[i]));
  }

  // ---- sum of the wavefronts' tiles: a lane holds, for token fr of each fragment, columns 4 fg .. 4 fg + 3 ----
  float* const red = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int a = 0; a < FA; ++a)
#pragma unroll
    for (int b = 0; b < FB; ++b)
      *reinterpret_cast<f32x4_t*>(red + (wave * RM + a * 16 + fr) * S::PITCH + b * 16 + fg * 4) = acc[a][b];
  __syncthreads();
  f32x4_t sum[QT];
#pragma unroll
  for (int q = 0; q < QT; ++q) {
    const int quad = q * 64 * W + tid;
    if (QUADS % (64 * W) && quad >= QUADS) continue;
    const float* src = red + (quad / (TN / 4)) * S::PITCH + (quad % (TN / 4)) * 4;
    sum[q] = *reinterpret_cast<const f32x4_t*>(src);
#pragma unroll
    for (int w = 1; w < W; ++w) sum[q] += *reinterpret_cast<const f32x4_t*>(src + w * RM * S::PITCH);
    if (S::PAIR)
#pragma unroll
      for (int w = 0; w < W; ++w) sum[q] += *reinterpret_cast<const f32x4_t*>(src + (w * RM + 8) * S::PITCH + 8);
  }

  if (EPI == EPI_SPLITK) {
    const int tile = tn * p.mt + tm, tiles = p.mt * p.nt;
    const rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(p.ws, 0, p.ksplit * tiles * QUADS * 16, 0x00020000);
#pragma unroll
    for (int q = 0; q < QT; ++q) {
      const int quad = q * 64 * W + tid;
      if (QUADS % (64 * W) && quad >= QUADS) continue;
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, sum[q]), rw, ((z * tiles + tile) * QUADS + quad) * 16, 0, SC1);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    int* const ticket = reinterpret_cast<int*>(smem);   // (a second shared variable makes the compiler drain the ring before every fragment read)
    if (tid == 0) *ticket = __hip_atomic_fetch_add(p.tickets + tile, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (*ticket != p.ksplit - 1) return;
    if (tid == 0) __hip_atomic_store(p.tickets + tile, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next launch
    asm volatile("" ::: "memory");
#pragma unroll
    for (int q = 0; q < QT; ++q) {
      const int quad = q * 64 * W + tid;
      if (QUADS % (64 * W) && quad >= QUADS) continue;
      f32x4_t v[MAX_SLICES];   // all in flight together; what is beyond the last slice reads as zero
#pragma unroll
      for (int s = 0; s < MAX_SLICES; ++s)
        v[s] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rw, s < p.ksplit ? ((s * tiles + tile) * QUADS + quad) * 16 : OOB, 0, SC1));
      sum[q] = v[0];
#pragma unroll
      for (int s = 1; s < MAX_SLICES; ++s) sum[q] += v[s];
    }
  }

#pragma unroll
  for (int q = 0; q < QT; ++q) {
    const int quad = q * 64 * W + tid;
    if (QUADS % (64 * W) && quad >= QUADS) continue;
    const int m = m0 + quad / (TN / 4), n = n0 + (quad % (TN / 4)) * 4;
    if (m >= p.M || n >= p.N) continue;
    float c[4] = {sum[q][0], sum[q][1], sum[q][2], sum[q][3]};
    const size_t o = (size_t)m * p.N + n;
    if (EPI == EPI_GATE) {
      if (bad) *p.flag = 1;
      const float e[4] = {__uint_as_float(ev[q].x << 16), __uint_as_float(ev[q].x & 0xffff0000u),
                          __uint_as_float(ev[q].y << 16), __uint_as_float(ev[q].y & 0xffff0000u)};
      float h[4];
#pragma unroll
      for (int x = 0; x < 4; ++x) h[x] = c[x] * sigmoidf_fast(c[x]) * e[x];
      if (p.outG) *reinterpret_cast<uint2*>(p.outG + o) = pack4(c);
      *reinterpret_cast<uint2*>(p.outH + o) = pack4(h);
    } else {
      if (p.residual) {   // the layer's output joins the residual stream: added in fp32, rounded once
        const uint2 rv = *reinterpret_cast<const uint2*>(p.residual + o);
        c[0] += __uint_as_float(rv.x << 16); c[1] += __uint_as_float(rv.x & 0xffff0000u);
        c[2] += __uint_as_float(rv.y << 16); c[3] += __uint_as_float(rv.y & 0xffff0000u);
      }
      *reinterpret_cast<uint2*>(reinterpret_cast<bf16_t*>(p.C) + o) = pack4(c);
    }
  }
}

// ---- choice of the tile and of the K split ----------------------------------------------------------------------
// Token tile: the smallest of 16, 32, 64 that holds the batch, else tiles of 64.  Weight tile: the smallest of 16, 32,
// 64 rows that gives at most one workgroup per CU (the rings leave room for one): more workgroups than CUs make a
// second round, fewer leave CUs without requests.  Gate product, us, 16 / 32 / 64 rows: d_model 2048, d_ff 8192, 16
// tokens 10.7 / 8.2 / 12.2, 64 tokens 15.8 / 11.7 / 14.5, 128 tokens - / 18.8 / 14.2; 1024 x 4096, 16 tokens 4.5 / 4.6 / 8.0,
// 128 tokens 8.3 / 6.4 / 7.7, 256 tokens - / 10.4 / 7.9.
// K is cut where that still leaves at most one workgroup per CU and as many K tiles per slice as outweigh the exchange
// of the partial tiles (about 1.3 us): the more tokens, the longer a K tile takes.  Layer forward, us, least 64 / 32 / 16
// K tiles: 1024 x 4096, 16 tokens 11.3 / 11.0 / 11.0, 64 tokens 16.8 / 14.4 / 13.2; 1536 x 5120, 64 tokens 26.8 / 21.5 / 21.5.
// (Up to 8 tokens no product is cut: 2048 weight rows and fewer take tiles of 8, more are over 128 workgroups.)
struct DecodePlan { int fa, fb, mt, nt, ksplit; bool pair; };

// K of more than 2048 (the down product of the larger layers) only with 16 weight rows: 2048 x 8192, 256 tokens, 25.0 us
// with 32 against 24.2 on the few-row kernel.
bool decode_plan(int M, int N, int K, bool plain, bool may_split, size_t ws_bytes, DecodePlan* plan) {
  const int fa = M <= 16 ? 1 : M <= 32 ? 2 : 4, mt = (M + 16 * fa - 1) / (16 * fa);
  // Up to 8 tokens: 8 weight rows per workgroup, so that K needs no slices and no exchange (2 to 3 us of a launch) while the
  // weight tiles still give one workgroup per CU.  Layer forward, us, 16 weight rows in slices / 8: 2048 x 8192, 1 token 18.2 / 16.9,
  // 4 tokens 19.1 / 18.0, 8 tokens 19.2 / 18.6; 1536 x 5120, 2 tokens 12.7 / 11.3; 1024 x 4096, 1 token 9.9 / 9.2, 8 tokens 10.2 / 9.6;
  // 512 x 1536, 1 token 6.9 / 6.5.  From K of 832 on, 13 K tiles of 64 for 8 wavefronts: 64 x 128, 4 tokens 5.2 / 5.4, 64 x 192,
  // 6 tokens 5.2 / 5.4, 832 x 832, 7 tokens 6.4 / 6.2.  (Each workgroup reads all tokens' rows whole, so the gain shrinks with the
  // tokens.  16 wavefronts with 2 K tiles in flight 17.4, 8 with 5 17.1.)
  if (plain && M <= 8 && N <= 8 * 256 && N % 8 == 0 && K > 12 * BK) {
    *plan = {1, 1, 1, N / 8, 1, true};
    return true;
  }
  for (int fb = 1; fb <= (fa == 4 ? 4 : 2); fb *= 2) {
    const int nt = (N + 16 * fb - 1) / (16 * fb);
    const bool last = fa < 4 && fb == 2;      // wide weight matrices and few tokens: several rounds
    if ((int64_t)mt * nt > 256 && !last) continue;
    if (fa == 4 && fb > 1 && K > 2048) break;
    int ks = 1;   // (slices of at least 16 K tiles, 8 at most: none of them is empty)
    const int least = M <= 16 ? 32 : 16;
    while (may_split && ks < MAX_SLICES && mt * nt * ks * 2 <= 256 && K / BK / (ks * 2) >= least &&
           (size_t)mt * nt * ks * 2 * fa * fb * 1024 <= ws_bytes)
      ks *= 2;
    *plan = {fa, fb, mt, nt, ks, false};
    return true;
  }
  return false;
}

template <class S>
void launch(int epi, const GemmArgs& p, hipStream_t s) {
  const dim3 grid((unsigned)(p.mt * p.nt * p.ksplit)), block(64 * S::W);
  if (epi == EPI_GATE) hipLaunchKernelGGL((gemm_decode_kernel<S, EPI_GATE>), grid, block, 0, s, p);
  else if (p.ksplit > 1) hipLaunchKernelGGL((gemm_decode_kernel<S, EPI_SPLITK>), grid, block, 0, s, p);
  else hipLaunchKernelGGL((gemm_decode_kernel<S, EPI_BF16>), grid, block, 0, s, p);
}

}  // namespace

// Worth it while one round of its workgroups covers the product; beyond, the few-row kernel's and the large kernel's
// tiles load less per CU.  d_model 2048, d_ff 8192, gate + down product, us, this / few-row: 1 token 17.6 / 28.0,
// 32 tokens 21.1 / 29.6, 64 tokens 26.6 / 31.5, 128 tokens 35.4 / 37.2, 256 tokens 45.2 / 40.8; 1024 x 4096: 32 tokens
// 12.0 / 19.8, 256 tokens 21.1 / 27.1, 320 tokens 27.7 / 25.9; 512 x 1536: 512 tokens 14.2 / 19.4.
bool stem_gemm_decode_fits(int M, int N, int K) {
  DecodePlan pl;
  return M <= 512 && K % BK == 0 && N % 4 == 0 && decode_plan(M, N, K, false, false, 0, &pl);
}

void stem_route_decode(int M, int N, int K, int epi, int64_t ws_bytes, int32_t* route) {
  DecodePlan pl = {};
  decode_plan(M, N, K, epi == EPI_BF16, epi == EPI_BF16 && ws_bytes > 0, (size_t)ws_bytes, &pl);
  route[0] = ROUTE_DECODE; route[1] = pl.pair ? 8 : 16 * pl.fa; route[2] = pl.pair ? 8 : 16 * pl.fb; route[3] = pl.ksplit;
}

hipError_t stem_gemm_decode_bf16(stem_ctx* ctx, int kid, int epi, const GemmArgs& a, hipStream_t s) {
  if (a.M <= 0 || a.N <= 0 || a.K <= 0) return hipSuccess;
  const int64_t lim = 0x7fffffff;
  if ((int64_t)a.M * a.lda * 2 > lim || (int64_t)a.N * a.ldb * 2 > lim) return hipErrorInvalidValue;
  DecodePlan pl;
  if (!stem_gemm_decode_fits(a.M, a.N, a.K) ||
      !decode_plan(a.M, a.N, a.K, epi == EPI_BF16, epi == EPI_BF16 && a.ws && a.tickets, a.ws_bytes, &pl))
    return hipErrorInvalidValue;
  if (epi != EPI_GATE && epi != EPI_BF16) return hipErrorInvalidValue;
  GemmArgs p = a;
  p.mt = pl.mt; p.nt = pl.nt; p.ksplit = pl.ksplit;
  p.inv_mt = 1.0f / (float)p.mt;
  p.inv_per_z = 1.0f / (float)(p.mt * p.nt);
  ProfScope ps(ctx, kid, s);
  if (pl.pair) hipLaunchKernelGGL((gemm_decode_kernel<PairShape<8, 4>, EPI_BF16>), dim3((unsigned)p.nt), dim3(512), 0, s, p);
  else if (pl.fa == 1 && pl.fb == 1) launch<Shape<1, 1, 8, 4>>(epi, p, s);
  else if (pl.fa == 1) launch<Shape<1, 2, 4, 6>>(epi, p, s);
  else if (pl.fa == 2 && pl.fb == 1) launch<Shape<2, 1, 8, 3>>(epi, p, s);
  else if (pl.fa == 2) launch<Shape<2, 2, 4, 4>>(epi, p, s);
  else if (pl.fb == 1) launch<Shape<4, 1, 4, 3>>(epi, p, s);
  else if (pl.fb == 2) launch<Shape<4, 2, 4, 3>>(epi, p, s);
  else launch<Shape<4, 4, 4, 2>>(epi, p, s);
  return hipGetLastError();
}
