// Host-resident table: device-side copy of the distinct rows a batch needs, read
// straight from pinned host memory (each lane pulls 16 bytes over the host link).
#include "stem_internal.h"

namespace {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;

// The host link bounds this kernel (57 GB/s), as long as about 256 KB are requested at any time; a compute unit gets 5.3 GB/s
// whatever it asks for.  So 16 workgroups, whose wavefronts each take 1 KB pieces of the rows, 4 in flight.
//
// What matters besides is whom the kernel keeps waiting.  A compute unit's loads return in order, so a GEMM tile that shares
// its compute unit with a copy waits for the link with every K tile, and a round of tiles for the slowest of them: the
// workgroups therefore claim LDS that no tile of the large bf16 products can do without (two of them fit a compute unit), and
// the products of a chunk leave 32 compute units free (STEM_PF_CHUNK_TILES).  The fp32 products' tiles (32 and 64 KB) still share
// with a copy.  The contexts of a device share two copy streams (api.hip, STEM_PF_LONG), so 32 compute units at most are held.
// A copy that shares the compute units with the GEMM tiles, 32 workgroups, 65536 tokens of 2048 x 8192, calls in turn on three contexts /
// two / by itself: 6.40 / 5.80 / 4.85 ms; with compute units to itself and a copy stream per context 5.22 / 4.83 / 4.61, with one for all
// 4.13 / 4.14 / 4.62.
constexpr int COPY_WGS = 16, FLIGHT = 4;
constexpr int COPY_LDS = 65 * 1024;   // two fit 160 KB, one and the smallest tile of gemm_bf16.hip (96 KB) do not
constexpr int BATCH = 64;             // pieces whose rows a wavefront looks up at a time, one per lane

// pieces: n rows of row_pieces pieces, 64 vectors of 16 bytes each but for the last of a row
__global__ __launch_bounds__(256) void copy_rows_kernel(const u32x4_t* __restrict__ src, const int32_t* __restrict__ src_row,
                                                        const int32_t* __restrict__ dst_slot, uint32_t pieces, uint32_t row_vecs,
                                                        uint32_t row_pieces, u32x4_t* __restrict__ dst) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t waves = gridDim.x * 4, wave = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (wave >= pieces) return;
  // lane l: row, slot and first vector of piece first + l * waves
  auto look_up = [&](uint32_t first, int& s, int& d, uint32_t& at) {
    uint32_t p = first + lane * waves;
    p = p < pieces ? p : pieces - 1;
    const uint32_t row = p / row_pieces;
    at = (p - row * row_pieces) * 64;
    s = src_row[row];
    d = dst_slot[row];
  };
  int src_l, dst_l;
  uint32_t at_l;
  look_up(wave, src_l, dst_l, at_l);
  for (uint32_t first = wave; first < pieces; first += BATCH * waves) {
    int src_n, dst_n;   // the next batch's, meanwhile
    uint32_t at_n;
    look_up(first + BATCH * waves < pieces ? first + BATCH * waves : first, src_n, dst_n, at_n);
    for (int k = 0; k < BATCH && first + k * waves < pieces; k += FLIGHT) {
      u32x4_t v[FLIGHT];
#pragma unroll
      for (int u = 0; u < FLIGHT; ++u) {
        const uint32_t at = __builtin_amdgcn_readlane(at_l, k + u) + lane;
        v[u] = src[(size_t)__builtin_amdgcn_readlane(src_l, k + u) * row_vecs + (at < row_vecs ? at : row_vecs - 1)];
      }
#pragma unroll
      for (int u = 0; u < FLIGHT; ++u) {
        const uint32_t at = __builtin_amdgcn_readlane(at_l, k + u) + lane;
        if (at < row_vecs && first + (k + u) * waves < pieces)
          dst[(size_t)__builtin_amdgcn_readlane(dst_l, k + u) * row_vecs + at] = v[u];
      }
    }
    src_l = src_n; dst_l = dst_n; at_l = at_n;
  }
}

// The copy's lists and remap.  Three hipMemcpyAsync calls take 25 to 35 us (above 16 KB through a copy engine and a handover to the
// next kernel), in which the gate product of the same call takes every compute unit: the row copy, which needs some for itself,
// then waits for a round of its tiles.  1024 x 4096, by itself / in turn on two contexts, us, row copies that share compute units /
// behind three memcpys / behind this kernel: 6000 tokens 430 / 452 / 418 and 342 / 381 / 344; 8192 tokens 532 / 554 / 519 and 425 /
// 475 / 433.  2048 x 8192, 16 tokens by itself 62 / 62 / 57.
__global__ __launch_bounds__(256) void copy_lists_kernel(const int32_t* __restrict__ remap_host, int32_t* __restrict__ remap, int64_t T,
                                                         const int32_t* __restrict__ order_host, int32_t* __restrict__ order,
                                                         int64_t n, int64_t second) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < T + 2 * n; i += (int64_t)gridDim.x * 256) {
    if (i < T) { remap[i] = remap_host[i]; continue; }
    const int64_t k = i - T < n ? i - T : i - T - n + second;
    order[k] = order_host[k];
  }
}

}  // namespace

hipError_t stem_copy_lists_kernel(stem_ctx* ctx, const int32_t* remap_host, int32_t* remap, int64_t T, const int32_t* order_host,
                                  int32_t* order, int64_t n, int64_t second, hipStream_t s) {
  if (T + n <= 0) return hipSuccess;
  ProfScope ps(ctx, K_LIST_COPY, s);
  const int grid = (int)std::min<int64_t>((T + 2 * n + 255) / 256, 1024);
  hipLaunchKernelGGL(copy_lists_kernel, dim3(grid), dim3(256), 0, s, remap_host, remap, T, order_host, order, n, second);
  return hipGetLastError();
}

hipError_t stem_copy_rows_kernel(stem_ctx* ctx, const void* E_host, const int32_t* src_row, const int32_t* dst_slot,
                                 int64_t n, int64_t row_bytes, void* E_compact, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  ProfScope ps(ctx, K_ROW_COPY, s);
  const int64_t row_vecs = row_bytes / 16, row_pieces = (row_vecs + 63) / 64;
  const int64_t pieces = n * row_pieces;   // below 2^31: at most 2^30 rows, and what device memory holds in whole pieces
  const int grid = (int)std::min<int64_t>((pieces + 3) / 4, COPY_WGS);
  hipLaunchKernelGGL(copy_rows_kernel, dim3(grid), dim3(256), COPY_LDS, s, (const u32x4_t*)E_host, src_row, dst_slot,
                     (uint32_t)pieces, (uint32_t)row_vecs, (uint32_t)row_pieces, (u32x4_t*)E_compact);
  return hipGetLastError();
}
