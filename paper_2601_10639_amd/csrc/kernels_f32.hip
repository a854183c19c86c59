// fp32 path of the STEM layer (small exactness-oriented runs) and the stand-alone
// element-wise kernel H = SiLU(G) * E[ids].
#include "stem_internal.h"

namespace {

__device__ __forceinline__ float sigmoid_f(float z) { return 1.0f / (1.0f + expf(-z)); }
__device__ __forceinline__ int checked_id(const int32_t* ids, int64_t t, int E_rows, int32_t* flag) {
  int id = ids[t];
  if ((unsigned)id >= (unsigned)E_rows) {
    *flag = 1;
    id = id < 0 ? 0 : E_rows - 1;
  }
  return id;
}

// ---- fp32 products on the matrix cores -------------------------------------------------------------
// C[m,n] = sum_k Aop[m,k] * Bop[n,k] with v_mfma_f32_32x32x2_f32 (full fp32 products and sums).  Operands are
// K-contiguous ([rows,K], OP_KC) or rows-contiguous ([K,rows], OP_MC); dimensions are multiples of 4 except the
// token count, so every 16-byte piece is whole or absent.
//
// A workgroup computes a TS x TS tile whose K tiles (32 wide) its W wavefronts share out: wavefront w takes every W-th,
// for the whole tile, through a ring of D K tiles of its own in LDS, filled by direct loads in whole lines.  So the
// main loop has no barrier, a short K range is requested whole before anything waits, and the chain of dependent MFMAs
// (64 cycles each), which is what a small product waits for, is W times shorter.  The W partial tiles are added through
// LDS in wavefront order; the element-wise part of the layer runs on the sums, its inputs requested behind the first
// K tiles.
// MFMA j of a group of 8 k takes k = 4 h + j from lane half h, for both operands alike, so a lane's four values of a
// K-contiguous operand are one 16-byte LDS read; those of a rows-contiguous operand are four 4-byte reads.
//
// Bound by the MFMAs from about 1000 tokens of 512 x 2048 on (82 to 126 TFLOP/s of 153), below by the launch and the
// first loads.  Against four wavefronts on one K tile with a barrier per K tile and operands through registers, forward
// and backward: 128 tokens of 64 x 256 25.3 -> 24.1 us, 600 of 128 x 400 41 -> 32, 1000 of 256 x 1024 76 -> 56, 1000 of
// 512 x 2048 172 -> 150, 4096 of 1024 x 2048 951 -> 820.
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef __amdgpu_buffer_rsrc_t rsrc_t;
constexpr int KT = 32;                  // K tile
constexpr uint32_t OOB = 0x80000000u;   // a buffer offset beyond any window: reads as zero

__device__ __forceinline__ void lds_dma_16(rsrc_t rs, char* lds_dst, uint32_t off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)lds_dst, 16, off, 0, 0, 0);
}

// One operand's K tile: TS x KT floats in LDS, KC as TS rows of 128 bytes (16-byte chunk c of row r at slot
// c ^ (r >> 1): a fragment read's 16 rows touch all banks once), MC as KT rows of TS floats.  A load of 1 KB covers ROWS
// of these rows; its window starts at the first of them (operands may exceed 2 GiB), and the lanes outside the matrix
// are given an offset beyond it.  WIDE: rows so long that 8 of them exceed a window; each lane has a 64-bit address of
// its own and the pieces pass through registers.
template <int TS, int LOP, bool WIDE>
struct TileF32 {
  static constexpr int LOADS = TS * KT * 4 / 1024, CH = LOP == OP_KC ? 8 : TS / 4, ROWS = 64 / CH;   // CH: chunks per row
  const char* at;        // the next K tile's first row
  int64_t group, step;   // bytes from one load's rows to the next one's, from one of this wavefront's K tiles to its next
  int64_t lane_row;      // WIDE: bytes to this lane's row of a load
  uint32_t off[LOADS];
  static __device__ __forceinline__ int swz(int r) { return (r >> 1) & 7; }
  __device__ __forceinline__ void init(const float* p, int64_t ld, int rows, int row0, int lane, int wave, int waves) {
    const int64_t pitch = ld * 4, kt = LOP == OP_KC ? KT * 4 : KT * pitch;
    at = reinterpret_cast<const char*>(p + (LOP == OP_KC ? row0 * ld : row0)) + wave * kt;
    group = ROWS * pitch;
    step = waves * kt;
    lane_row = lane / CH * pitch;
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int r = i * ROWS + lane / CH, c = lane % CH;                         // row in LDS, chunk slot
      const uint32_t o = (WIDE ? 0 : (uint32_t)lane_row) + (uint32_t)((LOP == OP_KC ? c ^ swz(r) : c) << 4);
      off[i] = row0 + (LOP == OP_KC ? r : c * 4) < rows ? o : OOB;
    }
  }
  // the K tile that `at` points to, of which `left` k exist, into `tile`; `at` moves on
  __device__ __forceinline__ void request(int left, char* tile, int lane) {
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int r = i * ROWS + lane / CH, k = LOP == OP_KC ? ((lane % CH) ^ swz(r)) << 2 : r;
      const uint32_t o = k < left ? off[i] : OOB;
      if (WIDE) {
        f32x4_t v = {0.f, 0.f, 0.f, 0.f};
        if (o != OOB) v = *reinterpret_cast<const f32x4_t*>(at + i * group + lane_row + o);
        *reinterpret_cast<f32x4_t*>(tile + i * 1024 + lane * 16) = v;
      } else {
        const rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(at + i * group), 0, 0x7fffffff, 0x00020000);
        lds_dma_16(rs, tile + i * 1024, o);
      }
    }
    at += step;
  }
  // the lane's four k of group g (8 k of the tile), row `row`
  static __device__ __forceinline__ f32x4_t frag(const char* lds, int row, int half, int g) {
    if (LOP == OP_KC) return *reinterpret_cast<const f32x4_t*>(lds + row * 128 + ((((g * 2 + half) ^ swz(row)) & 7) << 4));
    f32x4_t v;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = *reinterpret_cast<const float*>(lds + ((g * 8 + half * 4 + j) * TS + row) * 4);
    return v;
  }
};

// Waits until at most min(younger, MOST) K tiles of LOADS loads each are outstanding; the count is an immediate.  It
// counts the K tiles alone, each of them exactly LOADS instructions: whatever else a wavefront has in flight, and however
// many instructions the compiler makes of it, only makes the wait longer.
template <int LOADS, int MOST>
__device__ __forceinline__ void wait_all_but(int younger) {
  if (MOST == 0 || younger >= MOST) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(MOST * LOADS) : "memory");
  else wait_all_but<LOADS, (MOST > 0 ? MOST - 1 : 0)>(younger);
}

template <int TS, int W, int D>
struct ShapeF32 {
  static constexpr int PITCH = TS + 4;                       // row of a partial tile in LDS (floats)
  static constexpr int RING = W * D * 2 * TS * KT * 4, RED = W * TS * PITCH * 4, LDS_BYTES = RING > RED ? RING : RED;
};

// tile `block` of a product; smem: ShapeF32::LDS_BYTES of LDS
template <int TS, int W, int D, int LA, int LB, int EPI, bool WIDE = false>
__device__ __forceinline__ void gemm_f32_tile(const GemmF32Args& p, int block, char* smem) {
  typedef TileF32<TS, LA, WIDE> TA;
  typedef TileF32<TS, LB, WIDE> TB;
  constexpr int NB = TS / 32, OPERAND = TS * KT * 4, SLOT = 2 * OPERAND, LOADS = TA::LOADS + TB::LOADS;
  constexpr int PITCH = ShapeF32<TS, W, D>::PITCH;
  constexpr int QUADS = TS * TS / 4, QT = (QUADS + 64 * W - 1) / (64 * W), LPR = TS / 4;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ntn = (p.N - 1) / TS + 1;
  const int tm = block / ntn, tn = block - tm * ntn;
  const int m0 = tm * TS, n0 = tn * TS;
  const int r = lane & 31, half = lane >> 5;
  // rows and columns of this thread's quads, clamped into the matrix for the loads
  int ids_q[QT], mq[QT], nq[QT];
#pragma unroll
  for (int q = 0; q < QT; ++q) {
    const int quad = q * 64 * W + tid, m = m0 + quad / LPR, n = n0 + (quad % LPR) * 4;
    mq[q] = m < p.M ? m : p.M - 1;
    nq[q] = n < p.N ? n : 0;
    ids_q[q] = EPI == EPI_F32 ? 0 : p.ids[mq[q]];
  }
  TA ta;
  TB tb;
  ta.init(p.A, p.lda, p.M, m0, lane, wave, W);
  tb.init(p.B, p.ldb, p.N, n0, lane, wave, W);
  const int nk = (p.K - 1) / KT + 1;
  const int nw = nk > wave ? (nk - wave + W - 1) / W : 0;    // this wavefront's K tiles
  char* const ring = smem + wave * (D * SLOT);
  auto request = [&](int i, int slot) __attribute__((always_inline)) {
    const int left = p.K - (wave + i * W) * KT;
    ta.request(left, ring + slot * SLOT, lane);
    tb.request(left, ring + slot * SLOT + OPERAND, lane);
  };
  f32x4_t ev[QT], gv[QT];
  bool bad = false;
  // Younger than the first D K tiles and older than the rest; the barriers keep them in this place.
  auto load_inputs = [&]() __attribute__((always_inline)) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < QT; ++q) {
      asm volatile("" : "+v"(ids_q[q]));   // keeps what follows behind the requests
      int id = ids_q[q];
      bad |= (unsigned)id >= (unsigned)p.E_rows;   // reported to the host below, clamped so no access leaves the table
      id = id < 0 ? 0 : id < p.E_rows ? id : p.E_rows - 1;
      ev[q] = *reinterpret_cast<const f32x4_t*>(p.E + (int64_t)id * p.N + nq[q]);
      if (EPI == EPI_DH) gv[q] = *reinterpret_cast<const f32x4_t*>(p.inG + (int64_t)mq[q] * p.N + nq[q]);
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  // the usual case apart: behind conditional requests the compiler waits for all of them before it uses the ids
  if (nw >= D) {
#pragma unroll
    for (int d = 0; d < D; ++d) request(d, d);
    if (EPI != EPI_F32) load_inputs();
  } else {
#pragma unroll
    for (int d = 0; d < D - 1; ++d)
      if (d < nw) request(d, d);
    if (EPI != EPI_F32) load_inputs();
  }
  f32x16_t acc[NB][NB];
#pragma unroll
  for (int a = 0; a < NB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[a][b][e] = 0.f;
  int slot = 0;
  for (int i = 0; i < nw; ++i) {
    wait_all_but<LOADS, D - 1>(nw - 1 - i);
    const char* const st = ring + slot * SLOT;
    // the fragments of group g + 1 are read before the MFMAs of group g
    f32x4_t fa[2][NB], fb[2][NB];
    auto read = [&](int g) __attribute__((always_inline)) {
#pragma unroll
      for (int a = 0; a < NB; ++a) {
        fa[g & 1][a] = TA::frag(st, a * 32 + r, half, g);
        fb[g & 1][a] = TB::frag(st + OPERAND, a * 32 + r, half, g);
      }
    };
    read(0);
#pragma unroll
    for (int g = 0; g < KT / 8; ++g) {
      __builtin_amdgcn_sched_barrier(0);
      if (g + 1 < KT / 8) {
        read(g + 1);
      } else {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the slot has been read: it may be filled again
        if (i + D < nw) request(i + D, slot);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int a = 0; a < NB; ++a)
#pragma unroll
          for (int b = 0; b < NB; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[g & 1][b][j], fa[g & 1][a][j], acc[a][b], 0, 0, 0);
    }
    slot = slot + 1 == D ? 0 : slot + 1;
  }
  asm volatile("s_barrier" ::: "memory");                // nothing lands in LDS any more: every K tile has been waited for
  // partial tiles: a lane holds, for row r of each 32x32 piece, columns 8 g + 4 half .. + 3
  float* const red = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int a = 0; a < NB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<f32x4_t*>(red + (wave * TS + a * 32 + r) * PITCH + b * 32 + g * 8 + half * 4) =
            f32x4_t{acc[a][b][4 * g], acc[a][b][4 * g + 1], acc[a][b][4 * g + 2], acc[a][b][4 * g + 3]};
  __syncthreads();
#pragma unroll
  for (int q = 0; q < QT; ++q) {
    const int quad = q * 64 * W + tid;
    const int m = m0 + quad / LPR, n = n0 + (quad % LPR) * 4;
    if (QUADS % (64 * W) && quad >= QUADS) continue;
    if (m >= p.M || n >= p.N) continue;
    const float* src = red + (quad / LPR) * PITCH + (quad % LPR) * 4;
    f32x4_t c = *reinterpret_cast<const f32x4_t*>(src);
#pragma unroll
    for (int w = 1; w < W; ++w) c += *reinterpret_cast<const f32x4_t*>(src + w * TS * PITCH);
    const int64_t o = (int64_t)m * p.N + n;
    if (EPI == EPI_F32) {
      if (p.add) c += *reinterpret_cast<const f32x4_t*>(p.add + o);   // may be C itself: read before it is written
      *reinterpret_cast<f32x4_t*>(p.C + o) = c;
    } else {
      if (bad) *p.flag = 1;
      const f32x4_t e = ev[q];
      f32x4_t x, y;
      if (EPI == EPI_GATE) {        // G (optional) and H = SiLU(G) * E
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = c[j] * sigmoid_f(c[j]) * e[j];
        if (p.C) *reinterpret_cast<f32x4_t*>(p.C + o) = c;
        *reinterpret_cast<f32x4_t*>(p.out0 + o) = x;
      } else {                      // dU = dH * SiLU(G), dG = dH * E * SiLU'(G)
        const f32x4_t g = gv[q];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float s = sigmoid_f(g[j]);
          x[j] = c[j] * (g[j] * s);
          y[j] = c[j] * e[j] * (s * (1.0f + g[j] * (1.0f - s)));
        }
        *reinterpret_cast<f32x4_t*>(p.out0 + o) = x;
        *reinterpret_cast<f32x4_t*>(p.out1 + o) = y;
      }
    }
  }
}

template <int TS, int W, int D, int LA, int LB, int EPI>
__global__ __launch_bounds__(64 * W) void gemm_f32_kernel(GemmF32Args p) {
  __shared__ __attribute__((aligned(16))) char smem[ShapeF32<TS, W, D>::LDS_BYTES];
  gemm_f32_tile<TS, W, D, LA, LB, EPI>(p, blockIdx.x, smem);
}

// Rows of 2^26 elements and more, or more tiles than one launch takes (at most 4096 workgroups walk the tiles).  Bound by
// one load after another where the long dimension is summed over: 35 tokens of 8 x 67108868, forward and backward, 3.8 s.
template <int LA, int LB, int EPI>
__global__ __launch_bounds__(256) void gemm_f32_wide_kernel(GemmF32Args p, int tiles) {
  __shared__ __attribute__((aligned(16))) char smem[ShapeF32<32, 4, 1>::LDS_BYTES];
  for (int b = blockIdx.x; b < tiles; b += gridDim.x) {
    gemm_f32_tile<32, 4, 1, LA, LB, EPI, true>(p, b, smem);
    __syncthreads();   // the partial tiles have been read
  }
}

// The products of a backward pass that wait for nothing but dG, in one launch: dx first, the longest sum.  One after
// another they leave CUs idle three times over (1000 tokens, 256 x 1024: 256 workgroups each where 512 to 1024 fit, 11.5 +
// 10.7 + 10.8 us against 22.0; 128 tokens of 64 x 256, three launches against one, 6.5 + 6.4 + 6.1 against 6.3).
struct GradArgs { GemmF32Args dx, w[2]; int n_dx, n_w0; };
template <int D>
__global__ __launch_bounds__(256) void grads_f32_kernel(GradArgs p) {
  __shared__ __attribute__((aligned(16))) char smem[ShapeF32<32, 4, D>::LDS_BYTES];
  const int b = blockIdx.x;
  if (b < p.n_dx) {
    gemm_f32_tile<32, 4, D, OP_KC, OP_MC, EPI_F32>(p.dx, b, smem);
  } else {
    const int second = b - p.n_dx >= p.n_w0;
    gemm_f32_tile<32, 4, D, OP_MC, OP_MC, EPI_F32>(second ? p.w[1] : p.w[0], b - p.n_dx - (second ? p.n_w0 : 0), smem);
  }
}

// fp32: one thread per 4 features of one token.
__global__ void silu_gather_f32_kernel(const float* __restrict__ G, const int32_t* __restrict__ ids,
                                       const float* __restrict__ E, int E_rows, float* __restrict__ H,
                                       int64_t T, int F, int32_t* flag) {
  const int F4 = F >> 2;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= T * F4) return;
  const int64_t t = i / F4;
  const int c = (int)(i - t * F4) * 4;
  const int id = checked_id(ids, t, E_rows, flag);
  const float4 g = *reinterpret_cast<const float4*>(G + t * F + c);
  const float4 e = *reinterpret_cast<const float4*>(E + (int64_t)id * F + c);
  float4 h;
  h.x = g.x * sigmoid_f(g.x) * e.x; h.y = g.y * sigmoid_f(g.y) * e.y;
  h.z = g.z * sigmoid_f(g.z) * e.z; h.w = g.w * sigmoid_f(g.w) * e.w;
  *reinterpret_cast<float4*>(H + t * F + c) = h;
}

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;

// bf16: one workgroup per token, 16 bytes (8 features) per thread per sweep; the
// gathered row and the activation row are both read as full contiguous rows.
__global__ __launch_bounds__(256) void silu_gather_bf16_kernel(const bf16_t* __restrict__ G,
                                                               const int32_t* __restrict__ ids,
                                                               const bf16_t* __restrict__ E, int E_rows,
                                                               bf16_t* __restrict__ H, int64_t T, int F,
                                                               int32_t* flag) {
  for (int64_t t = blockIdx.x; t < T; t += gridDim.x) {
    const int id = checked_id(ids, t, E_rows, flag);
    const bf16_t* g = G + t * F;
    const bf16_t* e = E + (int64_t)id * F;
    bf16_t* h = H + t * F;
    for (int c = threadIdx.x * 8; c < F; c += blockDim.x * 8) {
      const uint4 gv = *reinterpret_cast<const uint4*>(g + c);
      const uint4 ev = *reinterpret_cast<const uint4*>(e + c);
      const uint32_t gw[4] = {gv.x, gv.y, gv.z, gv.w};
      const uint32_t ew[4] = {ev.x, ev.y, ev.z, ev.w};
      bf16x8_t out;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float g0 = __uint_as_float(gw[q] << 16), g1 = __uint_as_float(gw[q] & 0xffff0000u);
        const float e0 = __uint_as_float(ew[q] << 16), e1 = __uint_as_float(ew[q] & 0xffff0000u);
        out[2 * q] = (__bf16)(g0 * __builtin_amdgcn_rcpf(1.0f + __expf(-g0)) * e0);
        out[2 * q + 1] = (__bf16)(g1 * __builtin_amdgcn_rcpf(1.0f + __expf(-g1)) * e1);
      }
      *reinterpret_cast<bf16x8_t*>(h + c) = out;
    }
  }
}

}  // namespace

// Zero fill by a kernel rather than hipMemsetAsync, so that every call of the library can be recorded
// into a HIP graph (memset nodes have replayed wrongly on this platform).
__global__ __launch_bounds__(256) void fill_zero_kernel(uint32_t* __restrict__ p, size_t words) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < words; i += (size_t)gridDim.x * 256) p[i] = 0u;
}
hipError_t stem_fill_zero(void* p, size_t bytes, hipStream_t s) {   // bytes is a multiple of 4
  if (bytes == 0) return hipSuccess;
  const size_t words = bytes / 4;
  const unsigned grid = (unsigned)std::min<size_t>((words + 255) / 256, 2048);
  hipLaunchKernelGGL(fill_zero_kernel, dim3(grid), dim3(256), 0, s, static_cast<uint32_t*>(p), words);
  return hipGetLastError();
}

static int64_t tiles_f32(const GemmF32Args& p, int ts) { return (int64_t)((p.M - 1) / ts + 1) * ((p.N - 1) / ts + 1); }
static bool wide_f32(const GemmF32Args& p) { return std::max(p.lda, p.ldb) >= (1 << 26); }   // 8 rows of an operand exceed a 2 GiB window

// Up to here each product alone is at most one round of workgroups, two per CU; beyond, a launch each fills the chip and
// may take the larger tiles.  Forward and backward, us, three launches / one: 600 tokens of 128 x 400 32.5 / 21.2, 1000 of
// 256 x 1024 56 / 50, 2000 of 256 x 800 86 / 79.
constexpr int64_t GRADS_MAX_TILES = 512;
bool stem_grads_f32_fits(const GemmF32Args* dx, const GemmF32Args& w0, const GemmF32Args& w1) {
  auto small = [](const GemmF32Args& p) { return tiles_f32(p, 32) <= GRADS_MAX_TILES && !wide_f32(p); };
  return (!dx || small(*dx)) && small(w0) && small(w1);
}

hipError_t stem_grads_f32(stem_ctx* ctx, const GemmF32Args* dx, const GemmF32Args& w0, const GemmF32Args& w1, hipStream_t s) {
  GradArgs g = {};
  if (dx) { g.dx = *dx; g.n_dx = (int)tiles_f32(*dx, 32); }
  g.w[0] = w0; g.w[1] = w1;
  g.n_w0 = (int)tiles_f32(w0, 32);
  ProfScope ps(ctx, K_GRADS_F32, s);
  const unsigned n = (unsigned)(g.n_dx + g.n_w0 + tiles_f32(w1, 32));
  if (n <= 512) hipLaunchKernelGGL(grads_f32_kernel<2>, dim3(n), dim3(256), 0, s, g);   // K tiles in flight: as for a product by itself
  else hipLaunchKernelGGL(grads_f32_kernel<1>, dim3(n), dim3(256), 0, s, g);
  return hipGetLastError();
}

template <int LA, int LB, int EPI>
static void launch_f32(const GemmF32Args& p, hipStream_t s) {
  // 64x64 tiles where rounds of two workgroups per CU come out nearly full; else 32x32, two K tiles in flight per
  // wavefront (two workgroups per CU) up to 512 of them and one (four per CU) beyond.  us, 64x64 / 32x32 one / two in flight:
  // gate 1000 x 256 x 1024 12.9 / 11.8 / 13.1, down 22.3 / 12.8 / 10.8; gate 2048 x 512 x 1536 (768 tiles of 64) 44.9 / 40.7 / 42.4;
  // 4096 x 1024 x 2048 gate 151 / 154 / 176, down 137 / 146 / 156, dW 129 / 138 / 147.
  const int64_t t64 = tiles_f32(p, 64), t32 = tiles_f32(p, 32);
  const int64_t full64 = (t64 + 511) / 512 * 512;
  const bool large = t64 * 10 >= full64 * 9;
  if (wide_f32(p) || (large ? t64 : t32) >= (1 << 24))   // a launch has fewer than 2^32 threads
    hipLaunchKernelGGL((gemm_f32_wide_kernel<LA, LB, EPI>), dim3((unsigned)std::min<int64_t>(t32, 4096)), dim3(256), 0, s, p, (int)t32);
  else if (large)
    hipLaunchKernelGGL((gemm_f32_kernel<64, 4, 1, LA, LB, EPI>), dim3((unsigned)t64), dim3(256), 0, s, p);
  else if (t32 <= 512)
    hipLaunchKernelGGL((gemm_f32_kernel<32, 4, 2, LA, LB, EPI>), dim3((unsigned)t32), dim3(256), 0, s, p);
  else
    hipLaunchKernelGGL((gemm_f32_kernel<32, 4, 1, LA, LB, EPI>), dim3((unsigned)t32), dim3(256), 0, s, p);
}

hipError_t stem_gemm_f32(stem_ctx* ctx, int kid, int la, int lb, int epi, const GemmF32Args& p, hipStream_t s) {
  if (p.M <= 0 || p.N <= 0) return hipSuccess;
  ProfScope ps(ctx, kid, s);
  if (la == OP_KC && lb == OP_KC && epi == EPI_F32) launch_f32<OP_KC, OP_KC, EPI_F32>(p, s);
  else if (la == OP_KC && lb == OP_KC && epi == EPI_GATE) launch_f32<OP_KC, OP_KC, EPI_GATE>(p, s);
  else if (la == OP_KC && lb == OP_MC && epi == EPI_F32) launch_f32<OP_KC, OP_MC, EPI_F32>(p, s);
  else if (la == OP_KC && lb == OP_MC && epi == EPI_DH) launch_f32<OP_KC, OP_MC, EPI_DH>(p, s);
  else if (la == OP_MC && lb == OP_MC && epi == EPI_F32) launch_f32<OP_MC, OP_MC, EPI_F32>(p, s);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t stem_silu_gather(stem_ctx* ctx, int is_bf16, const void* G, const int32_t* ids, const void* E,
                            int E_rows, void* H, int64_t T, int F, hipStream_t s) {
  if (T <= 0) return hipSuccess;
  ProfScope ps(ctx, K_SILU_GATHER, s);
  if (is_bf16) {
    const int grid = (int)(T < 65536 ? T : 65536);
    hipLaunchKernelGGL(silu_gather_bf16_kernel, dim3(grid), dim3(256), 0, s, (const bf16_t*)G, ids,
                       (const bf16_t*)E, E_rows, (bf16_t*)H, T, F, ctx->flag);
  } else {
    const int64_t n = T * (F / 4);
    hipLaunchKernelGGL(silu_gather_f32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                       (const float*)G, ids, (const float*)E, E_rows, (float*)H, T, F, ctx->flag);
  }
  return hipGetLastError();
}
