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
// Workgroup = 4 wavefronts and a TS x TS tile.  TS = 64: each wavefront a 32x32 quadrant, K in tiles of 32.
// TS = 32: all four share the 32x32 tile and take a quarter of each 64-wide K tile, summed through LDS in a fixed
// order; four times the workgroups, and a quarter of the serial chain of MFMAs (64 cycles each), which is what a
// small product waits for.  Tiles travel global -> registers -> LDS, four K tiles in flight in registers (a short K
// range is requested whole before anything waits), two stages in LDS, one barrier per K tile.
// MFMA j of a group of 8 k takes k = 4 h + j from lane half h, for both operands alike, so a lane's four values of a
// K-contiguous operand are one 16-byte LDS read; those of a rows-contiguous operand are four 4-byte reads.
// The element-wise part of the layer runs in the epilogue, on rows read back from LDS.
//
// Against a 64x64 tile of scalar FMAs on 4-byte loads with nothing in flight across barriers, plus separate
// element-wise kernels: d_model 64, d_ff 256, 128 tokens 13-47 us -> 4-5 us per product; d_model 256, d_ff 1024, 1000 tokens
// 55-215 us -> 12-15 us.
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;

template <int TS, int LOP>
struct TileF32 {
  static constexpr int KT = TS == 64 ? 32 : 64;     // K tile: 8 KB of one operand either way
  static constexpr int ITEMS = 2;                   // 16-byte pieces per thread and K tile
  const float* p;                                   // the piece's address at K tile 0
  int64_t step;                                     // elements from one K tile to the next
  int64_t dist;                                     // from piece 0 to piece 1
  uint32_t lds0, lds1;
  int k_of[ITEMS];
  bool in[ITEMS];
  __device__ __forceinline__ void init(const float* base, int64_t ld, int rows, int row0, int tid) {
    if (LOP == OP_KC) {
      constexpr int CH = KT / 4;
      const int c = tid % CH, r = tid / CH;
      constexpr int RSTEP = 256 / CH;
      p = base + (int64_t)(row0 + r) * ld + c * 4;
      step = KT;
      dist = (int64_t)RSTEP * ld;
      k_of[0] = k_of[1] = c * 4;
      in[0] = row0 + r < rows;
      in[1] = row0 + r + RSTEP < rows;
      lds0 = slot(r, c);
      lds1 = slot(r + RSTEP, c);
    } else {
      constexpr int CH = TS / 4;
      const int c = tid % CH, k = tid / CH;
      constexpr int KSTEP = 256 / CH;
      p = base + (int64_t)k * ld + row0 + c * 4;
      step = (int64_t)KT * ld;
      dist = (int64_t)KSTEP * ld;
      k_of[0] = k;
      k_of[1] = k + KSTEP;
      in[0] = in[1] = row0 + c * 4 < rows;
      lds0 = (uint32_t)(k * TS + c * 4) * 4;
      lds1 = (uint32_t)((k + KSTEP) * TS + c * 4) * 4;
    }
  }
  // K-contiguous: 16-byte piece c of row r; the swizzle spreads a fragment read's 16 rows over all banks
  static __device__ __forceinline__ uint32_t slot(int r, int c) {
    return (uint32_t)(r * KT * 4 + ((c ^ (TS == 64 ? (r >> 1) & 7 : r & 15)) << 4));
  }
  __device__ __forceinline__ void load(int t, int K, f32x4_t (&v)[ITEMS]) const {
    const float* q = p + t * step;
    v[0] = v[1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if (in[0] && t * KT + k_of[0] < K) v[0] = *reinterpret_cast<const f32x4_t*>(q);
    if (in[1] && t * KT + k_of[1] < K) v[1] = *reinterpret_cast<const f32x4_t*>(q + dist);
  }
  __device__ __forceinline__ void store(char* lds, const f32x4_t (&v)[ITEMS]) const {
    *reinterpret_cast<f32x4_t*>(lds + lds0) = v[0];
    *reinterpret_cast<f32x4_t*>(lds + lds1) = v[1];
  }
  // the lane's four k of group g (8 k of the tile), row `row`
  static __device__ __forceinline__ f32x4_t frag(const char* lds, int row, int half, int g) {
    if (LOP == OP_KC) return *reinterpret_cast<const f32x4_t*>(lds + slot(row, g * 2 + half));
    f32x4_t v;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = *reinterpret_cast<const float*>(lds + ((g * 8 + half * 4 + j) * TS + row) * 4);
    return v;
  }
};

template <int TS, int LA, int LB, int EPI>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmF32Args p) {
  typedef TileF32<TS, LA> TA;
  typedef TileF32<TS, LB> TB;
  constexpr int KT = TA::KT, STAGE = 2 * TS * KT * 4;        // A and B of one K tile: 16 KB
  constexpr int DEPTH = 4;
  constexpr int PITCH = TS + 4;                              // epilogue row in LDS (floats)
  constexpr int PARTS = TS == 64 ? 1 : 4;                    // K quarters to sum
  constexpr int EPI_BYTES = PARTS * TS * PITCH * 4;
  __shared__ __attribute__((aligned(16))) char smem[EPI_BYTES > 2 * STAGE ? EPI_BYTES : 2 * STAGE];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ntn = (p.N + TS - 1) / TS;
  const int tm = blockIdx.x / ntn, tn = blockIdx.x - tm * ntn;
  const int m0 = tm * TS, n0 = tn * TS;
  const int wm = TS == 64 ? (wave >> 1) * 32 : 0, wn = TS == 64 ? (wave & 1) * 32 : 0;
  const int r = lane & 31, half = lane >> 5;
  TA ta;
  TB tb;
  ta.init(p.A, p.lda, p.M, m0, tid);
  tb.init(p.B, p.ldb, p.N, n0, tid);
  f32x16_t acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  f32x4_t ra[DEPTH][2], rb[DEPTH][2];
  const int nk = (p.K + KT - 1) / KT;
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) {
    ta.load(d, p.K, ra[d]);
    tb.load(d, p.K, rb[d]);
  }
  for (int t0 = 0; t0 < nk; t0 += DEPTH) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      if (t0 + d < nk) {
        char* st = smem + (d & 1) * STAGE;
        ta.store(st, ra[d]);
        tb.store(st + TS * KT * 4, rb[d]);
        ta.load(t0 + d + DEPTH, p.K, ra[d]);
        tb.load(t0 + d + DEPTH, p.K, rb[d]);
        __syncthreads();
        const int g0 = TS == 64 ? 0 : wave * 2, gn = TS == 64 ? 4 : 2;
#pragma unroll
        for (int g = 0; g < gn; ++g) {
          const f32x4_t fa = TA::frag(st, wm + r, half, g0 + g);
          const f32x4_t fb = TB::frag(st + TS * KT * 4, wn + r, half, g0 + g);
#pragma unroll
          for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[j], fa[j], acc, 0, 0, 0);
        }
      }
    }
  }
  __syncthreads();
  // lane holds, for row r of its 32x32 piece, columns 8 g + 4 half .. + 3
  {
    float* o = reinterpret_cast<float*>(smem) + (TS == 64 ? 0 : wave * TS * PITCH) + (wm + r) * PITCH + wn + half * 4;
#pragma unroll
    for (int g = 0; g < 4; ++g) *reinterpret_cast<f32x4_t*>(o + g * 8) = f32x4_t{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < TS * TS / 1024; ++it) {
    constexpr int LPR = TS / 4;
    const int row = it * (256 / LPR) + tid / LPR, col = (tid % LPR) * 4;
    const int m = m0 + row, n = n0 + col;
    if (m >= p.M || n >= p.N) continue;
    const float* src = reinterpret_cast<const float*>(smem) + row * PITCH + col;
    f32x4_t c = *reinterpret_cast<const f32x4_t*>(src);
#pragma unroll
    for (int q = 1; q < PARTS; ++q) c += *reinterpret_cast<const f32x4_t*>(src + q * TS * PITCH);
    const int64_t o = (int64_t)m * p.N + n;
    if (EPI == EPI_F32) {
      if (p.add) c += *reinterpret_cast<const f32x4_t*>(p.add + o);   // may be C itself: read before it is written
      *reinterpret_cast<f32x4_t*>(p.C + o) = c;
    } else {
      const int id = checked_id(p.ids, m, p.E_rows, p.flag);
      const f32x4_t e = *reinterpret_cast<const f32x4_t*>(p.E + (int64_t)id * p.N + n);
      f32x4_t x, y;
      if (EPI == EPI_GATE) {        // G (optional) and H = SiLU(G) * E
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = c[q] * sigmoid_f(c[q]) * e[q];
        if (p.C) *reinterpret_cast<f32x4_t*>(p.C + o) = c;
        *reinterpret_cast<f32x4_t*>(p.out0 + o) = x;
      } else {                      // dU = dH * SiLU(G), dG = dH * E * SiLU'(G)
        const f32x4_t g = *reinterpret_cast<const f32x4_t*>(p.inG + o);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float s = sigmoid_f(g[q]);
          x[q] = c[q] * (g[q] * s);
          y[q] = c[q] * e[q] * (s * (1.0f + g[q] * (1.0f - s)));
        }
        *reinterpret_cast<f32x4_t*>(p.out0 + o) = x;
        *reinterpret_cast<f32x4_t*>(p.out1 + o) = y;
      }
    }
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

template <int LA, int LB, int EPI>
static void launch_f32(const GemmF32Args& p, hipStream_t s) {
  // 64x64 tiles once they fill the chip (gate / down product, us, 64x64 and 32x32 tiles: 128 tokens of 64 x 256
  // 8.0, 11.0 and 6.6, 6.8; 1000 of 256 x 1024 15.3, 29.8 and 13.6, 14.7; 1000 of 512 x 2048 32.7, 56.0 and 33.5, 33.1;
  // 4096 of 1024 x 2048 182, 174 and 190, 183)
  const int64_t t64 = (int64_t)((p.M + 63) / 64) * ((p.N + 63) / 64), t32 = (int64_t)((p.M + 31) / 32) * ((p.N + 31) / 32);
  if (t64 >= 256) hipLaunchKernelGGL((gemm_f32_kernel<64, LA, LB, EPI>), dim3((unsigned)t64), dim3(256), 0, s, p);
  else hipLaunchKernelGGL((gemm_f32_kernel<32, LA, LB, EPI>), dim3((unsigned)t32), dim3(256), 0, s, p);
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
