// Gradient of the per-layer table, restricted to the rows a batch touches:
// stable sort of (token id, position) by counting ranks, by buckets of the vocabulary or by radix passes (in LDS, as merged runs, or digit by digit), distinct ids with run offsets, and a
// fixed-order segmented sum of the per-token row gradients.  Integer results are unique,
// floating sums use one fixed association, so every run gives the same bits.
#include <algorithm>

#include "stem_internal.h"

namespace {

constexpr int RADIX_BITS = 6;          // one digit value per lane of a wavefront
constexpr int RADIX = 1 << RADIX_BITS;
constexpr int SORT_WAVES = 16;         // wavefronts per workgroup
constexpr int KEYS_PER_WAVE = 256;     // 4 rounds of 64
constexpr int SORT_TILE = SORT_WAVES * KEYS_PER_WAVE;

__device__ __forceinline__ int load_key(const int32_t* __restrict__ keys, int64_t i, int V, int first_pass,
                                        int32_t* flag) {
  int k = keys[i];
  if (first_pass && (unsigned)k >= (unsigned)V) {
    *flag = 1;
    k = k < 0 ? 0 : V - 1;
  }
  return k;
}

// counts[d * nW + gw] = number of keys with digit d among wavefront gw's 256 keys
__global__ __launch_bounds__(1024) void sort_count_kernel(const int32_t* __restrict__ keys, int64_t T, int V,
                                                          int shift, int first_pass, int nW,
                                                          int32_t* __restrict__ counts, int32_t* flag) {
  __shared__ int hist[SORT_WAVES][RADIX];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int gw = blockIdx.x * SORT_WAVES + wave;
  hist[wave][lane] = 0;
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int r = 0; r < KEYS_PER_WAVE / 64; ++r) {
    const int64_t i = (int64_t)gw * KEYS_PER_WAVE + r * 64 + lane;
    if (i < T) {
      const int d = (load_key(keys, i, V, first_pass, flag) >> shift) & (RADIX - 1);
      atomicAdd(&hist[wave][d], 1);
    }
  }
  __builtin_amdgcn_wave_barrier();
  if (gw < nW) counts[lane * nW + gw] = hist[wave][lane];
}

// in-place exclusive scan of n ints by one workgroup of 1024 threads
__global__ __launch_bounds__(1024) void scan_kernel(int32_t* __restrict__ a, int n) {
  __shared__ int wsum[16];
  __shared__ int carry_s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = (n + 1023) / 1024;
  const int b = tid * per, e = min(n, b + per);
  int s = 0;
  for (int i = b; i < e; ++i) s += a[i];
  int inc = s;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(inc, o);
    if (lane >= o) inc += t;
  }
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  if (tid == 0) {
    int c = 0;
    for (int w = 0; w < 16; ++w) { const int t = wsum[w]; wsum[w] = c; c += t; }
    carry_s = c;
  }
  __syncthreads();
  int run = wsum[wave] + inc - s;
  for (int i = b; i < e; ++i) { const int t = a[i]; a[i] = run; run += t; }
}

// Stable scatter by digit.  Within a wavefront, a key's rank among equal digits of the
// same 64-key round comes from ballots; rounds and wavefronts are ordered by the scan.
__global__ __launch_bounds__(1024) void sort_scatter_kernel(const int32_t* __restrict__ keys,
                                                            const int32_t* __restrict__ vals, int64_t T, int V,
                                                            int shift, int first_pass, int nW,
                                                            const int32_t* __restrict__ counts,
                                                            int32_t* __restrict__ out_keys,
                                                            int32_t* __restrict__ out_vals, int32_t* flag) {
  __shared__ int base[SORT_WAVES][RADIX];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int gw = blockIdx.x * SORT_WAVES + wave;
  if (gw >= nW) return;
  base[wave][lane] = counts[lane * nW + gw];
  __builtin_amdgcn_wave_barrier();
  const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll 1
  for (int r = 0; r < KEYS_PER_WAVE / 64; ++r) {
    const int64_t i = (int64_t)gw * KEYS_PER_WAVE + r * 64 + lane;
    const bool valid = i < T;
    int key = 0, val = 0, d = 0;
    if (valid) {
      key = load_key(keys, i, V, first_pass, flag);
      val = first_pass ? (int)i : vals[i];
      d = (key >> shift) & (RADIX - 1);
    }
    uint64_t same = __ballot(valid);
#pragma unroll
    for (int b = 0; b < RADIX_BITS; ++b) {
      const bool bit = (d >> b) & 1;
      const uint64_t bb = __ballot(valid && bit);
      same &= bit ? bb : ~bb;
    }
    int pos = 0;
    if (valid) {
      const int rank = __popcll(same & below);
      pos = base[wave][d] + rank;
    }
    __builtin_amdgcn_wave_barrier();
    if (valid && (same & below) == 0) base[wave][d] += __popcll(same);
    __builtin_amdgcn_wave_barrier();
    if (valid) {
      out_keys[pos] = key;
      out_vals[pos] = val;
    }
  }
}

// Distinct ids, run offsets, and for every sorted position the index of its run.
constexpr int UNIQ_ITEMS = 8;
__global__ __launch_bounds__(1024) void unique_kernel(const int32_t* __restrict__ sorted, int64_t T,
                                                      int32_t* __restrict__ uniq_ids,
                                                      int32_t* __restrict__ seg_offsets,
                                                      int32_t* __restrict__ n_uniq, int32_t* __restrict__ seg_of) {
  __shared__ int wsum[16];
  __shared__ int total_s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int carry = 0;  // runs started before this sweep
  for (int64_t sweep = 0; sweep < T; sweep += 1024 * UNIQ_ITEMS) {
    const int64_t b = sweep + (int64_t)tid * UNIQ_ITEMS;
    int key[UNIQ_ITEMS];
    int prev = (b > 0 && b <= T) ? sorted[b - 1] : -1;
    int heads = 0;
    unsigned headmask = 0;
#pragma unroll
    for (int u = 0; u < UNIQ_ITEMS; ++u) {
      const int64_t k = b + u;
      if (k < T) {
        key[u] = sorted[k];
        const bool h = (k == 0) || key[u] != prev;
        prev = key[u];
        if (h) { ++heads; headmask |= 1u << u; }
      }
    }
    int inc = heads;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(inc, o);
      if (lane >= o) inc += t;
    }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    if (tid == 0) {
      int c = 0;
      for (int w = 0; w < 16; ++w) { const int t = wsum[w]; wsum[w] = c; c += t; }
      total_s = c;
    }
    __syncthreads();
    int run = carry + wsum[wave] + inc - heads;  // runs started before this thread's first item
#pragma unroll
    for (int u = 0; u < UNIQ_ITEMS; ++u) {
      const int64_t k = b + u;
      if (k < T) {
        if (headmask & (1u << u)) {
          uniq_ids[run] = key[u];
          seg_offsets[run] = (int)k;
          ++run;
        }
        seg_of[k] = run - 1;
      }
    }
    carry += total_s;
    __syncthreads();
  }
  if (tid == 0) {
    seg_offsets[carry] = (int)T;
    *n_uniq = carry;
  }
}


// ---- sort in LDS ------------------------------------------------------------------------
// The pair (id, position within the run) packs into one 32-bit key, so two LDS buffers hold a run of ITEMS * 1024
// keys, sorted by one workgroup.  The passes run over the id bits only; the position bits ride along and make the
// order total.  What bounds a pass is the instruction issue of one CU (6 ballots and a dozen more instructions per 64
// keys and round, rounds = ITEMS) and, below, the chain through the barriers; so the kernel comes in the sizes that
// occur, and a batch beyond the largest is cut into runs sorted side by side and merged by rank (below).
// Exclusive sum of v over the workgroup's threads in order; wsum: 16 ints of LDS.  The total goes to *total.
__device__ __forceinline__ int block_exclusive(int v, int* wsum, int lane, int wave, int* total = nullptr) {
  int inc = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(inc, o);
    if (lane >= o) inc += t;
  }
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    const int t = wsum[w];
    before += w < wave ? t : 0;
    all += t;
  }
  if (total) *total = all;
  return before + inc - v;
}

// RUNS: workgroup b sorts run b (keys [b * ITEMS * 1024, ...)) and writes only sorted_ids and perm (global positions).
template <int ITEMS, bool RUNS>
__global__ __launch_bounds__(1024) void sort_lds_kernel(const int32_t* __restrict__ ids, int T, int V, int pos_bits,
                                                        int passes, int32_t* __restrict__ sorted_ids,
                                                        int32_t* __restrict__ perm, int32_t* __restrict__ uniq_ids,
                                                        int32_t* __restrict__ seg_offsets, int32_t* __restrict__ n_uniq,
                                                        int32_t* __restrict__ seg_of, int32_t* flag) {
  __shared__ uint32_t buf[2][ITEMS * 1024];
  __shared__ int table[RADIX * SORT_WAVES];  // [digit][wave], scanned in place
  __shared__ __attribute__((aligned(16))) uint8_t cnt8[SORT_WAVES][RADIX][ITEMS < 4 ? 4 : ITEMS];
  __shared__ int wsum[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int first = RUNS ? blockIdx.x * ITEMS * 1024 : 0;
  const int n = min(T - first, ITEMS * 1024);
  const int per_wave = (n + SORT_WAVES - 1) / SORT_WAVES;      // contiguous keys per wavefront
  const int w0 = wave * per_wave, w1 = min(n, w0 + per_wave);
  const uint32_t pos_mask = (1u << pos_bits) - 1u;
  {
    int kv[ITEMS];
#pragma unroll
    for (int u = 0; u < ITEMS; ++u) kv[u] = (tid + 1024 * u) < n ? ids[first + tid + 1024 * u] : 0;
    bool bad = false;
#pragma unroll
    for (int u = 0; u < ITEMS; ++u) {
      const int i = tid + 1024 * u;
      int k = kv[u];
      if ((unsigned)k >= (unsigned)V) { bad = true; k = k < 0 ? 0 : V - 1; }
      if (i < n) buf[0][i] = ((uint32_t)k << pos_bits) | (uint32_t)i;
    }
    if (bad) *flag = 1;
  }
  __syncthreads();
  const uint64_t below = (1ull << lane) - 1ull;
  int cur = 0;
  // Per pass and wavefront: ITEMS rounds of 64 keys.  A key's rank among equal digits of its round
  // comes from ballots; the per-round digit counts go to cnt8[wave][digit][round] (bytes), lane d
  // then turns digit d's counts into running offsets, so no round waits for the one before.
  for (int p = 0; p < passes; ++p) {
    const int shift = pos_bits + p * RADIX_BITS;
    uint32_t key[ITEMS];
    uint32_t dr[ITEMS];  // digit | rank << 8 | valid << 16
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      const int i = w0 + r * 64 + lane;
      key[r] = i < w1 ? buf[cur][i] : 0u;
    }
    uint32_t* const mine = reinterpret_cast<uint32_t*>(&cnt8[wave][lane][0]);
#pragma unroll
    for (int x = 0; x < (ITEMS + 3) / 4; ++x) mine[x] = 0;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      const bool valid = (w0 + r * 64 + lane) < w1;
      const int d = (key[r] >> shift) & (RADIX - 1);
      uint64_t same = __ballot(valid);
#pragma unroll
      for (int b = 0; b < RADIX_BITS; ++b) {
        const bool bit = (d >> b) & 1;
        const uint64_t bb = __ballot(valid && bit);
        same &= bit ? bb : ~bb;
      }
      const int rank = __popcll(same & below);
      if (valid && rank == 0) cnt8[wave][d][r] = (uint8_t)__popcll(same);
      dr[r] = (uint32_t)d | ((uint32_t)rank << 8) | (valid ? 1u << 16 : 0u);
    }
    __builtin_amdgcn_wave_barrier();
    // lane = digit: running offsets over the rounds
    uint32_t cw[(ITEMS + 3) / 4];
#pragma unroll
    for (int x = 0; x < (ITEMS + 3) / 4; ++x) cw[x] = mine[x];
    int pre[ITEMS];
    int tot = 0;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      pre[r] = tot;
      tot += (int)((cw[r >> 2] >> ((r & 3) * 8)) & 0xffu);
    }
    table[lane * SORT_WAVES + wave] = tot;
    __syncthreads();
    table[tid] = block_exclusive(table[tid], wsum, lane, wave);   // 1024 entries, one per thread
    __syncthreads();
    const int base = table[lane * SORT_WAVES + wave];  // first output slot of (digit = lane, this wavefront)
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      const int d = dr[r] & 0xff;
      const int start = __shfl(base + pre[r], d);
      if (dr[r] >> 16) buf[cur ^ 1][start + (int)((dr[r] >> 8) & 0xff)] = key[r];
    }
    __syncthreads();
    cur ^= 1;
  }
  if (RUNS) {
#pragma unroll
    for (int u = 0; u < ITEMS; ++u) {
      const int k = tid + 1024 * u;
      if (k < n) {
        sorted_ids[first + k] = (int)(buf[cur][k] >> pos_bits);
        perm[first + k] = first + (int)(buf[cur][k] & pos_mask);
      }
    }
    return;
  }
  // Unpack and number the runs of equal ids, position k = u * 1024 + tid throughout (coalesced in global memory,
  // conflict-free in LDS).  A position's run index is the number of run heads at or before it, minus one: heads of
  // earlier (sweep, wavefront) pairs from a scanned table of ballot counts, heads of earlier lanes from the ballot.
  int* cnt = table;                     // [sweep * SORT_WAVES + wave], reused
  uint64_t headmask[ITEMS];
  int idv[ITEMS];
#pragma unroll
  for (int u = 0; u < ITEMS; ++u) {
    const int k = tid + 1024 * u;
    bool head = false;
    idv[u] = 0;
    if (k < n) {
      const uint32_t key = buf[cur][k];
      const int id = (int)(key >> pos_bits);
      idv[u] = id;
      sorted_ids[k] = id;
      perm[k] = (int)(key & pos_mask);
      head = (k == 0) || id != (int)(buf[cur][k - 1] >> pos_bits);
    }
    headmask[u] = __ballot(head);
    if (lane == 0) cnt[u * SORT_WAVES + wave] = __popcll(headmask[u]);
  }
  __syncthreads();
  {
    int total;
    const int v = tid < ITEMS * SORT_WAVES ? cnt[tid] : 0;
    const int before = block_exclusive(v, wsum, lane, wave, &total);
    if (tid < ITEMS * SORT_WAVES) cnt[tid] = before;
    if (tid == 0) {
      seg_offsets[total] = n;
      *n_uniq = total;
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < ITEMS; ++u) {
    const int k = tid + 1024 * u;
    if (k < n) {
      const bool head = (headmask[u] >> lane) & 1ull;
      const int run = cnt[u * SORT_WAVES + wave] + __popcll(headmask[u] & below) + (head ? 0 : -1);
      if (head) { uniq_ids[run] = idv[u]; seg_offsets[run] = k; }
      seg_of[k] = run;
    }
  }
}

// ---- up to 2048 ids: ranks by counting ----------------------------------------------------------------
// One workgroup's passes are a chain of barriers, and it has one compute unit of the chip.  Here each workgroup places 8 ids and
// looks at all of them: an id's place is the number of smaller (id, position) keys, counted by ballots, 64 keys a compare; where its run
// begins, the number of keys below (id, 0); the number of its run, the distinct ids below it, from a bitmap of the ids in LDS and its
// prefix sums.  Nothing passes between workgroups, so one launch does it all.  What bounds it is the launch, the id loads and
// four barriers.  us in a graph, before (one workgroup's passes) / this, Zipf ids: 128 ids 5.8 / 4.1, 1000 7.5 / 4.4, 1999 12.6 / 5.3.
// (16 ids a workgroup: 1000 ids 4.9, 1999 6.1; 32: 6.0 and 7.7.)  Counting is quadratic: 4096 ids 7.6, 8192 15.7.
constexpr int RANK_WORDS = 8192;                 // 32 KB of bitmap: vocabularies up to 2^18
constexpr int RANK_MAX = 2048;                   // ids
template <int CHUNKS, int OWN>                   // T <= CHUNKS * 1024; ids a workgroup places, at most a wavefront's lanes
__global__ __launch_bounds__(1024) void sort_ranks_kernel(const int32_t* __restrict__ ids, int T, int V, int pos_bits,
                                                          int32_t* __restrict__ sorted_ids, int32_t* __restrict__ perm,
                                                          int32_t* __restrict__ uniq_ids, int32_t* __restrict__ seg_offsets,
                                                          int32_t* __restrict__ n_uniq, int32_t* __restrict__ seg_of, int32_t* flag) {
  constexpr int WORDS = RANK_WORDS / 1024;       // per thread
  __shared__ __attribute__((aligned(16))) uint32_t bitmap[RANK_WORDS];
  __shared__ int pre[1024];                      // ids set before a thread's words
  __shared__ int counts[SORT_WAVES][OWN];
  __shared__ int wsum[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i0 = blockIdx.x * OWN, own_i = min(i0 + (lane & (OWN - 1)), T - 1);
  int kv[CHUNKS], own_id = ids[own_i];
#pragma unroll
  for (int c = 0; c < CHUNKS; ++c) kv[c] = tid + 1024 * c < T ? ids[tid + 1024 * c] : 0;
  for (int w = tid; w < (V + 31) / 32; w += 1024) bitmap[w] = 0;
  __syncthreads();
  auto clamped = [&](int id) { return (unsigned)id < (unsigned)V ? id : id < 0 ? 0 : V - 1; };
  own_id = clamped(own_id);
  uint32_t key[CHUNKS];
  bool bad = false;
#pragma unroll
  for (int c = 0; c < CHUNKS; ++c) {
    const int i = tid + 1024 * c, id = clamped(kv[c]);
    key[c] = 0xffffffffu;                        // beyond the batch: smaller than no key
    if (i < T) {
      bad |= id != kv[c];
      key[c] = ((uint32_t)id << pos_bits) | (uint32_t)i;
      // (a look first: a frequent id would queue all its lanes at one word)
      if (!(bitmap[id >> 5] >> (id & 31) & 1u)) atomicOr(&bitmap[id >> 5], 1u << (id & 31));
    }
  }
  if (bad) *flag = 1;
  const uint32_t own_key = ((uint32_t)own_id << pos_bits) | (uint32_t)own_i;
  int mine = 0;
#pragma unroll 2                                 // (unrolled whole, the compiler keeps all counts to the end, and spills)
  for (int q = 0; q < OWN; ++q) {
    const uint32_t k = __builtin_amdgcn_readlane(own_key, q), k_id = k >> pos_bits << pos_bits;
    int below = 0, start = 0;
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
      below += __popcll(__ballot(key[c] < k));
      start += __popcll(__ballot(key[c] < k_id));
    }
    mine = lane == q ? below | start << 16 : mine;   // sums over the wavefronts up to 2048 each
  }
  if (lane < OWN) counts[wave][lane] = mine;
  __syncthreads();                               // counts, and all ids are in the bitmap
  int set = 0, distinct;
  if (tid * WORDS * 32 < V)
#pragma unroll
    for (int x = 0; x < WORDS; ++x)
      if ((tid * WORDS + x) * 32 < V) set += __popc(bitmap[tid * WORDS + x]);
  pre[tid] = block_exclusive(set, wsum, lane, wave, &distinct);
  __syncthreads();
  if (blockIdx.x == 0 && tid == 0) {
    seg_offsets[distinct] = T;
    *n_uniq = distinct;
  }
  if (tid >= OWN || i0 + tid >= T) return;
  int sum = 0;
#pragma unroll
  for (int w = 0; w < SORT_WAVES; ++w) sum += counts[w][tid];
  const int place = sum & 0xffff, start = sum >> 16;
  const int word = own_id >> 5, first = word & ~(WORDS - 1);
  int run = pre[word / WORDS] + __popc(bitmap[word] & ((1u << (own_id & 31)) - 1u));
  for (int x = first; x < word; ++x) run += __popc(bitmap[x]);
  sorted_ids[place] = own_id;
  perm[place] = own_i;
  seg_of[place] = run;
  if (place == start) { uniq_ids[run] = own_id; seg_offsets[run] = start; }
}

// ---- more ids, up to 16384: a workgroup for every bucket of the vocabulary -------------------------------------------
// Merged runs are three launches.  Here each of up to 256 workgroups owns the ids of a stretch of the vocabulary: it looks at all ids, keeps
// its own in order in LDS and sorts them by one stable counting pass (a wavefront's rounds of 64 by ballots, a table of counts per wavefront
// and id, its scan, the rounds again).  Where its ids begin is the number of smaller ids, the number of its first run the distinct smaller
// ids, from a bitmap in LDS.  Nothing passes between workgroups, and one frequent id makes one workgroup's pass longer, not the others'.
// What bounds it are the looks at all ids and their bits in the bitmap.  us in a graph, before (ranks up to 8192 ids, then merged runs) / this,
// Zipf ids and one id for all: 3000 ids 7.6 / 7.1 and 7.8 / 7.4, 4096 7.8 / 7.3 and 7.9 / 7.9, 5000 14.9 / 8.2 and 15.2 / 9.6, 8192 15.9 /
// 9.2 and 16.0 / 11.4, 16384 24.6 / 13.5 and 22.0 / 19.7; 2048 ids 5.5 / 7.6 and 5.7 / 7.1.  (Rounds by bits alone, and twice: 16384 ids 15.0
// and 35.1.)  16384 ids are what its LDS holds.
constexpr int BUCKET_MIN = 2048, BUCKET_MAX = 16384;   // ids: more than the one, up to the other
constexpr int BUCKET_IDS = 1024;                 // vocabulary entries of a bucket at most
template <int CHUNKS>                            // T <= CHUNKS * 1024
__global__ __launch_bounds__(1024) void sort_buckets_kernel(const int32_t* __restrict__ ids, int T, int V, int R, int bits,
                                                            int32_t* __restrict__ sorted_ids, int32_t* __restrict__ perm,
                                                            int32_t* __restrict__ uniq_ids, int32_t* __restrict__ seg_offsets,
                                                            int32_t* __restrict__ n_uniq, int32_t* __restrict__ seg_of, int32_t* flag) {
  constexpr int POS = 14;                        // bits of a position
  __shared__ __attribute__((aligned(16))) uint32_t bitmap[RANK_WORDS];
  __shared__ uint32_t list[CHUNKS * 1024];       // id in the bucket << POS | position
  __shared__ uint16_t table[SORT_WAVES][BUCKET_IDS];
  __shared__ int bin_start[BUCKET_IDS], bin_run[BUCKET_IDS];
  __shared__ int own_s[CHUNKS * SORT_WAVES], less_s[SORT_WAVES], wsum[4][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lo = blockIdx.x * R, hi = min(lo + R, V);            // R: a multiple of 32
  const uint64_t below = (1ull << lane) - 1ull;
  int kv[CHUNKS];
#pragma unroll
  for (int c = 0; c < CHUNKS; ++c) kv[c] = ids[min(tid + 1024 * c, T - 1)];
  for (int w = tid; w < lo >> 5; w += 1024) bitmap[w] = 0;
  for (int w = 0; w < SORT_WAVES; ++w)
    if (tid < R) table[w][tid] = 0;
  int less = 0;
  uint64_t own[CHUNKS];
#pragma unroll
  for (int c = 0; c < CHUNKS; ++c) {
    const int id = min(max(kv[c], 0), V - 1);
    if (blockIdx.x == 0 && id != kv[c]) *flag = 1;
    kv[c] = tid + 1024 * c < T ? id : 0x7fffffff;                // beyond the batch: in no bucket
    less += __popcll(__ballot(kv[c] < lo));
    own[c] = __ballot(kv[c] >= lo && kv[c] < hi);
    if (lane == 0) own_s[c * SORT_WAVES + wave] = __popcll(own[c]);
  }
  if (lane == 0) less_s[wave] = less;
  __syncthreads();
  int n;
  {
    const int v = tid < CHUNKS * SORT_WAVES ? own_s[tid] : 0, before = block_exclusive(v, wsum[0], lane, wave, &n);
    if (tid < CHUNKS * SORT_WAVES) own_s[tid] = before;
  }
#pragma unroll
  for (int c = 0; c < CHUNKS; ++c)               // (a look first: a frequent id would queue all its lanes at one word)
    if (kv[c] < lo && !(bitmap[kv[c] >> 5] >> (kv[c] & 31) & 1u)) atomicOr(&bitmap[kv[c] >> 5], 1u << (kv[c] & 31));
  int base = 0;
#pragma unroll
  for (int w = 0; w < SORT_WAVES; ++w) base += less_s[w];
  __syncthreads();
#pragma unroll
  for (int c = 0; c < CHUNKS; ++c)
    if (own[c] >> lane & 1ull) list[own_s[c * SORT_WAVES + wave] + __popcll(own[c] & below)] = (uint32_t)(kv[c] - lo) << POS | (uint32_t)(tid + 1024 * c);
  int set = 0, distinct;
  for (int w = tid; w < lo >> 5; w += 1024) set += __popc(bitmap[w]);
  block_exclusive(set, wsum[1], lane, wave, &distinct);          // its barrier is the list's too

  // Every wavefront counts a stretch of the list by rounds of 64, and notes of each entry how many with its id are before it there.
  // Lanes with one id find each other by comparing with the first one's, a few times over (a frequent id fills whole rounds), then bit by bit.
  uint16_t* const nth = reinterpret_cast<uint16_t*>(bitmap);     // the bitmap has been counted
  static_assert(CHUNKS * 1024 * 2 <= sizeof(bitmap), "an entry each");
  const int stretch = ((n + 1023) >> 10) * 64;
  for (int i0 = wave * stretch; i0 < min((wave + 1) * stretch, n); i0 += 64) {
    const int i = i0 + lane;
    const bool valid = i < n;
    const int id = (int)(list[min(i, n - 1)] >> POS);
    uint64_t left = __ballot(valid), same = 0;
    for (int peel = 0; peel < 3 && left; ++peel) {
      const uint64_t m = __ballot(id == __builtin_amdgcn_readlane(id, __builtin_ctzll(left))) & left;
      if (m >> lane & 1ull) same = m;
      left &= ~m;
    }
    if (left) {
      uint64_t rest = left;
      for (int x = 0; x < bits; ++x) {
        const bool bit = (id >> x) & 1;
        const uint64_t bb = __ballot(bit);
        rest &= bit ? bb : ~bb;
      }
      if (left >> lane & 1ull) same = rest;
    }
    if (valid) {
      const int before = table[wave][id];
      nth[i] = (uint16_t)(before + __popcll(same & below));
      if (!(same & below)) table[wave][id] = (uint16_t)(before + __popcll(same));
    }
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  int count = 0;                                 // of id lo + tid; the table becomes what earlier wavefronts have of it
  if (tid < R)
    for (int w = 0; w < SORT_WAVES; ++w) {
      const int t = table[w][tid];
      table[w][tid] = (uint16_t)count;
      count += t;
    }
  int here;
  const int start = block_exclusive(count, wsum[2], lane, wave), run = distinct + block_exclusive(count > 0, wsum[3], lane, wave, &here);
  if (tid < R) {
    bin_start[tid] = base + start;
    bin_run[tid] = run;
    if (count > 0) { uniq_ids[run] = lo + tid; seg_offsets[run] = base + start; }
  }
  if (hi == V && tid == 0) {
    seg_offsets[distinct + here] = T;
    *n_uniq = distinct + here;
  }
  __syncthreads();
  for (int i = tid; i < n; i += 1024) {
    const int id = (int)(list[i] >> POS), place = bin_start[id] + table[i / stretch][id] + nth[i];
    sorted_ids[place] = lo + id;
    perm[place] = (int)(list[i] & ((1u << POS) - 1u));
    seg_of[place] = bin_run[id];
  }
}

// ---- larger batches: merge of the sorted runs by rank, then distinct ids and run index ---------------
// A key's place in the whole order is its place in its own run, plus, of every earlier run, the keys at most as large,
// plus, of every later run, the keys that are smaller: the merge is stable, needs no passes, and every key finds its
// place alone, 16 binary searches of L2-resident runs in flight at a time (64 neighbouring keys take nearly the same
// path through a run, so their loads coalesce).
constexpr int MERGE_WAYS = 16;
__global__ __launch_bounds__(256) void merge_runs_kernel(const int32_t* __restrict__ keys, const int32_t* __restrict__ vals,
                                                         int T, int R, int32_t* __restrict__ sorted_ids,
                                                         int32_t* __restrict__ perm) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  const int ic = min(i, T - 1);
  const int id = keys[ic], val = vals[ic];
  const int own = ic / R, nr = (T + R - 1) / R;
  int rank = ic - own * R;
  for (int q0 = 0; q0 < nr; q0 += MERGE_WAYS) {
    int pos[MERGE_WAYS], len[MERGE_WAYS];
#pragma unroll
    for (int x = 0; x < MERGE_WAYS; ++x) {
      const int q = q0 + x;
      pos[x] = 0;
      len[x] = q < nr && q != own ? min(R, T - q * R) : 0;
    }
    for (int step = R; step > 0; step >>= 1) {
      int k[MERGE_WAYS];
#pragma unroll
      for (int x = 0; x < MERGE_WAYS; ++x)
        k[x] = keys[min(q0 + x, nr - 1) * R + max(min(pos[x] + step, len[x]) - 1, 0)];
#pragma unroll
      for (int x = 0; x < MERGE_WAYS; ++x)
        if (pos[x] + step <= len[x] && k[x] < id + (q0 + x < own ? 1 : 0)) pos[x] += step;
    }
#pragma unroll
    for (int x = 0; x < MERGE_WAYS; ++x) rank += pos[x];
  }
  if (i < T) {
    sorted_ids[rank] = id;
    perm[rank] = val;
  }
}

// Distinct ids, run offsets and run index of 1024 sorted positions per workgroup, which counts the run heads before its
// own itself (T / 2 reads on average, from L2) instead of waiting for its predecessors.
__global__ __launch_bounds__(1024) void unique_blocks_kernel(const int32_t* __restrict__ sorted, int T,
                                                             int32_t* __restrict__ uniq_ids,
                                                             int32_t* __restrict__ seg_offsets,
                                                             int32_t* __restrict__ n_uniq, int32_t* __restrict__ seg_of) {
  __shared__ int wsum[2][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int k0 = blockIdx.x * 1024, k = k0 + tid;
  int key = 0;
  bool head = false;
  if (k < T) {
    key = sorted[k];
    head = k == 0 || sorted[k - 1] != key;
  }
  int mine = 0;
#pragma unroll 8
  for (int j = tid; j < k0; j += 1024) mine += j == 0 || sorted[j] != sorted[j - 1];
  int earlier, here;
  block_exclusive(mine, wsum[0], lane, wave, &earlier);
  const int run = earlier + block_exclusive(head ? 1 : 0, wsum[1], lane, wave, &here) - (head ? 0 : 1);
  if (k < T) {
    if (head) { uniq_ids[run] = key; seg_offsets[run] = k; }
    seg_of[k] = run;
  }
  if (tid == 0 && k0 + 1024 >= T) {
    seg_offsets[earlier + here] = T;
    *n_uniq = earlier + here;
  }
}

// ---- segmented sum -----------------------------------------------------------------
constexpr int SEG_ROWS = 32;  // sorted positions per chunk

template <bool BF16> struct RowVec;
template <> struct RowVec<true> {
  static constexpr int COLS = 8;
  typedef __attribute__((ext_vector_type(4))) uint32_t raw_t;
  static __device__ __forceinline__ raw_t load(const void* base, int64_t row, int F, int col) {
    return __builtin_nontemporal_load(reinterpret_cast<const raw_t*>(reinterpret_cast<const bf16_t*>(base) + row * F + col));
  }
  static __device__ __forceinline__ raw_t load_plain(const void* base, int64_t row, int F, int col) {
    return *reinterpret_cast<const raw_t*>(reinterpret_cast<const bf16_t*>(base) + row * F + col);
  }
  static __device__ __forceinline__ void add(const raw_t& v, float (&acc)[8]) {
    const uint32_t w[4] = {v[0], v[1], v[2], v[3]};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      acc[2 * q] += __uint_as_float(w[q] << 16);
      acc[2 * q + 1] += __uint_as_float(w[q] & 0xffff0000u);
    }
  }
};
template <> struct RowVec<false> {
  static constexpr int COLS = 4;
  typedef __attribute__((ext_vector_type(4))) float raw_t;
  static __device__ __forceinline__ raw_t load(const void* base, int64_t row, int F, int col) {
    return *reinterpret_cast<const raw_t*>(reinterpret_cast<const float*>(base) + row * F + col);
  }
  static __device__ __forceinline__ raw_t load_plain(const void* base, int64_t row, int F, int col) { return load(base, row, F, col); }
  static __device__ __forceinline__ void add(const raw_t& v, float (&acc)[4]) {
    acc[0] += v.x; acc[1] += v.y; acc[2] += v.z; acc[3] += v.w;
  }
};

template <int COLS>
__device__ __forceinline__ void store_cols(float* dst, const float (&a)[COLS]) {
#pragma unroll
  for (int q = 0; q < COLS; q += 4) *reinterpret_cast<float4*>(dst + q) = make_float4(a[q], a[q + 1], a[q + 2], a[q + 3]);
}

// One workgroup sums the rows of sorted positions [c*SEG_ROWS, (c+1)*SEG_ROWS) for a slab
// of 256*COLS columns, in ascending position.  A run that lies wholly inside the chunk
// is written to its output row; the (at most two) pieces of runs that cross the chunk's
// borders go to part[c][0] (piece holding the chunk's first position) or part[c][1].
// The chunk's row numbers and run indices are fetched once into LDS, so all row loads can
// be in flight together and run ends need no further global reads.
template <bool BF16>
__global__ __launch_bounds__(256) void seg_reduce_kernel(const void* __restrict__ dU,
                                                         const int32_t* __restrict__ perm,
                                                         const int32_t* __restrict__ seg_of, int64_t T, int F,
                                                         float* __restrict__ dE_rows,
                                                         float* __restrict__ part) {
  constexpr int COLS = RowVec<BF16>::COLS;
  __shared__ int s_perm[SEG_ROWS];
  __shared__ int s_seg[SEG_ROWS + 2];  // [0] = run of the position before the chunk, [n+1] = of the one after
  const int c = blockIdx.y;
  const int k0 = c * SEG_ROWS;
  const int k1 = (int)min((int64_t)k0 + SEG_ROWS, T);
  const int n = k1 - k0;
  const int tid = threadIdx.x;
  if (tid < n) s_perm[tid] = perm[k0 + tid];
  if (tid < n + 2) {
    const int64_t k = (int64_t)k0 - 1 + tid;
    s_seg[tid] = (k >= 0 && k < T) ? seg_of[k] : -1;
  }
  __syncthreads();
  const int col = (blockIdx.x * 256 + tid) * COLS;
  if (col >= F) return;
  const int first_seg = s_seg[1], last_seg = s_seg[n];
  const bool first_open = s_seg[0] == first_seg;      // the first run began before the chunk
  const bool last_open = s_seg[n + 1] == last_seg;    // the last run goes on after the chunk
  float acc[COLS];
#pragma unroll
  for (int q = 0; q < COLS; ++q) acc[q] = 0.f;
  int cur = first_seg;

  auto flush = [&](int j) {
    const bool open = (j == first_seg && first_open) || (j == last_seg && last_open);
    float* dst = open ? part + ((int64_t)c * 2 + (j == first_seg ? 0 : 1)) * F + col
                      : dE_rows + (int64_t)j * F + col;
    store_cols<COLS>(dst, acc);
  };

  // all of the chunk's row loads are requested before the first store: loads and stores return
  // through one in-order counter, so a load requested after a store is not seen before that store
  // has been acknowledged
  constexpr int UNR = SEG_ROWS;
#pragma unroll
  for (int kb = 0; kb < SEG_ROWS; kb += UNR) {
    typename RowVec<BF16>::raw_t data[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u)
      if (kb + u < n) data[u] = RowVec<BF16>::load(dU, s_perm[kb + u], F, col);
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      if (kb + u < n) {
        const int sg = s_seg[kb + u + 1];
        if (sg != cur) {
          flush(cur);
          cur = sg;
#pragma unroll
          for (int q = 0; q < COLS; ++q) acc[q] = 0.f;
        }
        RowVec<BF16>::add(data[u], acc);
      }
    }
  }
  flush(cur);
}

// The chunk in which a border-crossing run starts adds up that run's pieces: workgroup = that chunk
// and a slab of 64 * COLS columns; the run's pieces are cut into four consecutive stretches, one per
// wavefront, each summed in chunk order, and the four sums are added in order.  (One fixed
// association, so every run gives the same bits.  With one thread summing all of a run's pieces the
// most frequent id's 69 pieces were a chain of five dependent rounds of loads.)
template <int COLS>
__global__ __launch_bounds__(256) void seg_combine_kernel(const int32_t* __restrict__ seg_of,
                                                          const int32_t* __restrict__ seg_offsets, int64_t T,
                                                          int F, float* __restrict__ dE_rows,
                                                          const float* __restrict__ part) {
  __shared__ float red[3][64][COLS + 1];
  const int c = blockIdx.x;
  const int k0 = c * SEG_ROWS;
  const int64_t k1 = (int64_t)k0 + SEG_ROWS;
  if (k1 >= T) return;                                 // nothing after this chunk
  // the four run indices that decide whether this chunk has anything to do, requested together
  const int j = seg_of[k1 - 1], after = seg_of[k1], first = seg_of[k0], before = k0 > 0 ? seg_of[k0 - 1] : -1;
  if (after != j) return;                              // the last run ends with the chunk
  if (first == j && before == j) return;               // the run began in an earlier chunk
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = (blockIdx.y * 64 + lane) * COLS;
  const bool live = col < F;
  const int slot = (first == j) ? 0 : 1;
  const int hi = seg_offsets[j + 1];
  const int n = (hi - 1) / SEG_ROWS - c + 1;           // pieces: this chunk's, then slot 0 of the following chunks
  const int q = (n + 3) >> 2;
  const int p0 = wave * q, p1 = min(n, p0 + q);
  float acc[COLS];
#pragma unroll
  for (int x = 0; x < COLS; ++x) acc[x] = 0.f;
  if (live) {
    constexpr int UNR = 16;
    for (int pb = p0; pb < p1; pb += UNR) {
      float data[UNR][COLS];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        if (pb + u < p1) {
          const int pc = pb + u;
          const float* src = part + ((int64_t)(c + pc) * 2 + (pc == 0 ? slot : 0)) * F + col;
#pragma unroll
          for (int x = 0; x < COLS; x += 4) {
            const float4 v = *reinterpret_cast<const float4*>(src + x);
            data[u][x] = v.x; data[u][x + 1] = v.y; data[u][x + 2] = v.z; data[u][x + 3] = v.w;
          }
        }
      }
#pragma unroll
      for (int u = 0; u < UNR; ++u)
        if (pb + u < p1)
#pragma unroll
          for (int x = 0; x < COLS; ++x) acc[x] += data[u][x];
    }
  }
  if (wave > 0) {
#pragma unroll
    for (int x = 0; x < COLS; ++x) red[wave - 1][lane][x] = acc[x];
  }
  __syncthreads();
  if (wave == 0 && live) {
    for (int w = 1; w < 4; ++w)
      if (w * q < n)
#pragma unroll
        for (int x = 0; x < COLS; ++x) acc[x] += red[w - 1][lane][x];
    store_cols<COLS>(dE_rows + (int64_t)j * F + col, acc);
  }
}

// Small batches, where a chunk's row loads and the second launch are all latency: whole runs are summed in one launch, with a
// workgroup for every position and band of up to 16 slabs of 64 * COLS columns.  A run is summed by the workgroups of its first
// positions, the others end at once.
//
// A run of up to 16 rows is one round of loads of one wavefront for each slab, which the wavefronts of the run's first workgroup share out.
// Longer ones are dealt to 4 * PARTS row groups, PARTS = 1, 2, 4, 8 up to 64, 128, 256 rows and beyond, in which PARTS teams of four
// wavefronts take 1 / PARTS of a slab's columns each: a lane then has 16 rows at most (32 of 1024, 64 of 2048), and a long run is read
// by as many more compute units: the run's workgroups take its (slab, part) pairs in turn.  Rows are added in ascending position, four
// at a time, then the groups of a wavefront in order, then the wavefronts: no term of 1024 meets more than 20 additions.
// us in a graph, sums of a sorted batch: two launches of 32-row chunks / a workgroup for every position and slab / now:
//                    bf16 1024 x 4096     bf16 256 x 8192      fp32 1024 x 2048     fp32 256 x 1024     bf16 1999 x 8192
//   Zipf ids         11.6 / 8.0 / 6.7     11.3 / 5.1 / 5.1     12.6 / 6.9 / 5.0     12.0 / 3.0 / 3.0    17.7 / 18.0 / 14.3
//   one id for half  12.0 / 7.2 / 6.1     11.2 / 5.9 / 6.2     12.7 / 6.0 / 4.9     12.1 / 4.0 / 4.0    17.3 / - / 12.6
//   one id for all   10.6 / 8.3 / 7.4     10.4 / 6.4 / 6.3      8.7 / 9.2 / 5.8      8.0 / 5.1 / 5.1    13.8 / 19.7 / 14.0
// (a workgroup of four wavefronts for a long run's whole slab: 58.5 at 1024 x 4096, one id for all.)
// The relative error of fp32 unit normals, all of one id, 1024 rows: 1.20e-7 in two launches, 2.92e-7 with four wavefronts for the
// whole run, 1.04e-7 so.
// (Row loads that bypass the caches, as the large batches' do: one id for all, bf16 1024 x 4096 15.5 us instead of 8.2.)
constexpr int ROUND = 16;        // rows a lane requests together

template <bool BF16>
__device__ __forceinline__ void add_quad(const typename RowVec<BF16>::raw_t* rows, int n, float (&acc)[RowVec<BF16>::COLS]) {
  constexpr int COLS = RowVec<BF16>::COLS;
  if (n <= 0) return;
  float t[COLS];
#pragma unroll
  for (int x = 0; x < COLS; ++x) t[x] = 0.f;
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (u < n) RowVec<BF16>::add(rows[u], t);
#pragma unroll
  for (int x = 0; x < COLS; ++x) acc[x] += t[x];
}

// Adds `rows` (at most R) rows of a run of n, from its r-th on.  Loads carry no conditions, or the compiler waits for those it
// cannot count; what lies beyond the rows is read for nothing, within the run.
template <bool BF16, int R, class Rows>
__device__ __forceinline__ void add_rows(const void* dU, Rows perm, int r, int rows, int n, int F, int col,
                                         float (&acc)[RowVec<BF16>::COLS]) {
  int row[R];
  typename RowVec<BF16>::raw_t data[R];
#pragma unroll
  for (int u = 0; u < R; ++u) row[u] = perm[min(r + u, n - 1)];
#pragma unroll
  for (int u = 0; u < R; ++u) data[u] = RowVec<BF16>::load_plain(dU, row[u], F, col);
#pragma unroll
  for (int u = 0; u < R; u += 4) add_quad<BF16>(data + u, rows - u, acc);
}

// Slabs of a band at most: a run of more than 64, 128, 256 rows then has as many workgroups as (slab, part) pairs, one each.
constexpr int MAX_BAND = 16;

// a run of n rows is summed in 1 << run_shift(n) parts of a slab's columns
__device__ __forceinline__ int run_shift(int n) { return n <= 4 * ROUND ? 0 : n <= 8 * ROUND ? 1 : n <= 16 * ROUND ? 2 : 3; }

// Up to ROUND rows of a run, from its r-th on, in the columns of a wavefront's lane.
template <bool BF16, class Rows>
__device__ __forceinline__ void add_round(const void* dU, Rows rows_of, int r, int rows, int F, int col, float (&acc)[RowVec<BF16>::COLS]) {
  typename RowVec<BF16>::raw_t data[ROUND];
#pragma unroll
  for (int u = 0; u < ROUND; ++u)
    if (u < rows) data[u] = RowVec<BF16>::load_plain(dU, rows_of[r + u], F, col);
#pragma unroll
  for (int u = 0; u < ROUND; ++u) asm("" : "+v"(data[u]));   // or additions move to the loads, and wait there for each by itself
#pragma unroll
  for (int u = 0; u < ROUND; u += 4) add_quad<BF16>(data + u, rows - u, acc);
}

// A run of up to ROUND rows, in a slab's columns, by one wavefront
template <bool BF16, class Rows>
__device__ __forceinline__ void sum_short(const void* dU, Rows rows_of, int n, int slab, int lane, int F, float* out) {
  constexpr int COLS = RowVec<BF16>::COLS;
  const int col = (slab * 64 + lane) * COLS;
  float acc[COLS];
#pragma unroll
  for (int x = 0; x < COLS; ++x) acc[x] = 0.f;
  add_round<BF16>(dU, rows_of, 0, n, F, col < F ? col : 0, acc);
  if (col < F) store_cols<COLS>(out + col, acc);
}

// The same for up to 4 rows and 4 slabs, `step` apart, all requested together
template <bool BF16, class Rows>
__device__ __forceinline__ void sum_shortest(const void* dU, Rows rows_of, int n, int slab, int step, int slabs, int lane, int F, float* out) {
  constexpr int COLS = RowVec<BF16>::COLS, STEPS = ROUND / 4;
  typename RowVec<BF16>::raw_t data[STEPS][4];
#pragma unroll
  for (int s = 0; s < STEPS; ++s)
    if (slab + s * step < slabs) {
      const int col = ((slab + s * step) * 64 + lane) * COLS, colc = col < F ? col : 0;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (u < n) data[s][u] = RowVec<BF16>::load_plain(dU, rows_of[u], F, colc);
    }
#pragma unroll
  for (int s = 0; s < STEPS; ++s)
#pragma unroll
    for (int u = 0; u < 4; ++u) asm("" : "+v"(data[s][u]));
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    const int col = ((slab + s * step) * 64 + lane) * COLS;
    float acc[COLS];
#pragma unroll
    for (int x = 0; x < COLS; ++x) acc[x] = 0.f;
    add_quad<BF16>(data[s], n, acc);
    if (slab + s * step < slabs && col < F) store_cols<COLS>(out + col, acc);
  }
}

// A part of a longer run's slab by four wavefronts, t their thread, red 256 * (COLS + 1) floats: first the row groups' sums, then, behind
// a barrier, all of them.
template <bool BF16, class Rows>
__device__ __forceinline__ void sum_groups(const void* dU, Rows rows_of, int n, int part, int slab, int t, int F, float* red,
                                           float (&acc)[RowVec<BF16>::COLS]) {
  constexpr int COLS = RowVec<BF16>::COLS;
  const int shift = run_shift(n);
#pragma unroll
  for (int x = 0; x < COLS; ++x) acc[x] = 0.f;
  if (shift == 0) {   // rows of whole wavefronts: their numbers come through scalar loads
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int q = (n + 3) >> 2, r = wave * q, rows = min(q, n - r);
    const int col = (slab * 64 + (t & 63)) * COLS;
    add_round<BF16>(dU, rows_of, r, rows, F, col < F ? col : 0, acc);
  } else {
    const int width = 64 >> shift, groups = 4 << shift;    // lanes of a part, row groups
    const int col = (slab * 64 + part * width + (t & (width - 1))) * COLS, colc = col < F ? col : 0;
    const int q = (n + groups - 1) >> (2 + shift);         // rows of a group (the last ones may have fewer, or none)
    const int r = (t >> (6 - shift)) * q, rows = min(q, n - r);
    if (q <= ROUND / 2) add_rows<BF16, ROUND / 2>(dU, rows_of, r, rows, n, F, colc, acc);
    else
      for (int rb = 0; rb < q; rb += ROUND) add_rows<BF16, ROUND>(dU, rows_of, r + rb, rows - rb, n, F, colc, acc);
  }
#pragma unroll
  for (int x = 0; x < COLS; ++x) red[t * (COLS + 1) + x] = acc[x];
}
template <bool BF16>
__device__ __forceinline__ void sum_join(int n, int part, int slab, int t, int F, const float* red, float (&acc)[RowVec<BF16>::COLS],
                                         float* out) {
  constexpr int COLS = RowVec<BF16>::COLS;
  const int shift = run_shift(n);
  if (shift == 0) {
    const int col = (slab * 64 + t) * COLS;
    if (t >= 64 || col >= F) return;
    for (int w = 1; w < 4; ++w)
#pragma unroll
      for (int x = 0; x < COLS; ++x) acc[x] += red[(w * 64 + t) * (COLS + 1) + x];
    store_cols<COLS>(out + col, acc);
    return;
  }
  // a column: the groups of each wavefront in order, then the wavefronts
  const int width = 64 >> shift, first_col = (slab * 64 + part * width) * COLS;
  for (int c = t; c < width * COLS && first_col + c < F; c += 256) {
    const float* from = red + (c / COLS) * (COLS + 1) + c % COLS;
    float sum = 0.f;
    for (int w = 0; w < 4; ++w) {
      float s = 0.f;
      for (int g = 0; g < 1 << shift; ++g) s += from[(w * 64 + g * width) * (COLS + 1)];
      sum += s;
    }
    out[first_col + c] = sum;
  }
}

// The slabs of the workgroup's band, and whether the rank-th workgroup of a run of n rows has any of its sums.
template <bool BF16>
__device__ __forceinline__ int band_slabs(int F, int band) {
  constexpr int COLS = RowVec<BF16>::COLS;
  return min((F + 64 * COLS - 1) / (64 * COLS) - (int)blockIdx.y * band, band);
}
template <int GROUPS>
__device__ __forceinline__ bool sums_some(int n, int rank, int slabs) {
  return rank == 0 || (n > ROUND && rank * GROUPS < slabs << run_shift(n));
}

// That workgroup's sums: GROUPS teams of four wavefronts.  rows_of: the run's positions in the batch; out: its row.
template <bool BF16, int GROUPS, class Rows>
__device__ __forceinline__ void sum_run(const void* dU, Rows rows_of, int n, int rank, int slabs, int slab0, int F, float* out,
                                        float* red) {
  constexpr int COLS = RowVec<BF16>::COLS;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (n <= 4) {   // (slabs counted from the row's start)
    for (int slab = slab0 + wave; slab < slab0 + slabs; slab += 4 * GROUPS * (ROUND / 4))
      sum_shortest<BF16>(dU, rows_of, n, slab, 4 * GROUPS, slab0 + slabs, lane, F, out);
    return;
  }
  if (n <= ROUND) {
    for (int slab = wave; slab < slabs; slab += 4 * GROUPS) sum_short<BF16>(dU, rows_of, n, slab0 + slab, lane, F, out);
    return;
  }
  const int team = wave >> 2, t = tid & 255, shift = run_shift(n), item = rank * GROUPS + team;
  const int slab = item >> shift, part = item & ((1 << shift) - 1);
  const bool mine = slab < slabs;
  float acc[COLS];
  red += team * 256 * (COLS + 1);
  if (mine) sum_groups<BF16>(dU, rows_of, n, part, slab0 + slab, t, F, red, acc);
  __syncthreads();
  if (mine) sum_join<BF16>(n, part, slab0 + slab, t, F, red, acc, out);
}

template <bool BF16, int GROUPS>
__global__ __launch_bounds__(256 * GROUPS) void seg_runs_kernel(const void* __restrict__ dU, const int32_t* __restrict__ perm,
                                                                const int32_t* __restrict__ seg_of,
                                                                const int32_t* __restrict__ seg_offsets, int F, int band,
                                                                float* __restrict__ dE_rows) {
  __shared__ float red[GROUPS * 256 * (RowVec<BF16>::COLS + 1)];   // a thread's sums, one float apart
  const int k = blockIdx.x, slabs = band_slabs<BF16>(F, band), most = (slabs * 8 + GROUPS - 1) / GROUPS;   // workgroups of a run
  const int j = seg_of[k], far = seg_of[max(k - most, 0)];
  if (k >= most && far == j) return;
  const int start = seg_offsets[j], n = seg_offsets[j + 1] - start;
  if (sums_some<GROUPS>(n, k - start, slabs))
    sum_run<BF16, GROUPS>(dU, perm + start, n, k - start, slabs, blockIdx.y * band, F, dE_rows + (int64_t)j * F, red);
}

// The same for a batch that is not sorted yet, with the sort: every workgroup looks at all ids.  The tokens with its token's id are the
// run, the number of smaller ids is where the run begins, and the number of distinct smaller ids, from a bitmap of the ids in LDS, the run's
// number.  The workgroup of a run's first token writes the sort's outputs for the run besides.  Nothing passes between
// workgroups.
// What bounds it is the launch, the ids' loads and three barriers, beyond some 1500 tokens the looks at all ids by every workgroup.  us in
// a graph, rank sort and sums as two launches / this, Zipf ids: fp32 128 x 256 7.0 / 4.2, 1000 x 1024 9.5 / 6.8, 2048 x 2048 16.5 / 11.9; bf16
// 128 x 8192 8.8 / 5.5, 512 x 8192 12.7 / 7.3, 1024 x 4096 13.1 / 9.0, 1999 x 8192 23.2 / 19.4, 2048 x 4096 19.7 / 13.8; one id for all:
// fp32 1000 x 1024 9.6 / 8.5, 2048 x 256 13.9 / 13.1, bf16 2000 x 1536 16.1 / 15.5.  (One slab of a short run after another 1999 x 8192
// 20.7, 2048 x 4096 14.9; counting with the ballots of every 64 ids for rank
// and run, not only of those that hold the id: 1000 x 1024 7.8, 1999 x 8192 22.1; a workgroup for every token and slab: 1000 x 1024 11.3.)
constexpr int SMALL_MAX = 2048;                  // tokens
constexpr int SMALL_WORDS = 4096;                // 16 KB of bitmap: vocabularies up to 2^17
template <bool BF16, int GROUPS, int MOST>       // GROUPS of four wavefronts; up to MOST tokens
__global__ __launch_bounds__(256 * GROUPS) void sort_sum_kernel(const int32_t* __restrict__ ids, int T, int V,
                                                                const void* __restrict__ dU, int F, int band, int32_t* __restrict__ sorted_ids,
                                                                int32_t* __restrict__ perm, int32_t* __restrict__ uniq_ids,
                                                                int32_t* __restrict__ seg_offsets, int32_t* __restrict__ n_uniq,
                                                                int32_t* __restrict__ seg_of, float* __restrict__ dE_rows, int32_t* flag) {
  constexpr int COLS = RowVec<BF16>::COLS, THREADS = 256 * GROUPS, WAVES = 4 * GROUPS, CHUNKS = MOST / THREADS;
  __shared__ float red[GROUPS * 256 * (COLS + 1)];
  __shared__ uint32_t bitmap[SMALL_WORDS];
  __shared__ uint64_t same_s[MOST / 64];         // which of 64 tokens have the id
  __shared__ int rows[MOST];                     // the run's tokens
  __shared__ uint64_t counts[WAVES];             // smaller ids | earlier tokens of the run << 16 | its tokens << 32
  __shared__ int set_s[WAVES];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = blockIdx.x;
  const bool total = i == 0;                     // also looks for ids outside the table, and counts all distinct ones
  auto clamped = [&](int id) { return min(max(id, 0), V - 1); };
  int kv[CHUNKS];
#pragma unroll
  for (int c = 0; c < CHUNKS; ++c) kv[c] = ids[min(tid + THREADS * c, T - 1)];
  const int own = clamped(ids[i]);
  int less = 0, early = 0, n = 0;
#pragma unroll
  for (int c = 0; c < CHUNKS; ++c) {
    const int id = clamped(kv[c]), at = (c * WAVES + wave) * 64;
    if (total && id != kv[c]) *flag = 1;
    kv[c] = at + lane < T ? id : 0x7fffffff;     // beyond the batch: no id
    less += __popcll(__ballot(kv[c] < own));
    const uint64_t same = __ballot(kv[c] == own);
    if (same) {                                  // (few of the wavefronts' chunks: the scalar unit is what counting waits for)
      n += __popcll(same);
      early += __popcll(i >= at + 64 ? same : i > at ? same & ((1ull << (i - at)) - 1ull) : 0ull);
    }
  }
  if (lane == 0) counts[wave] = (uint32_t)(less + (early << 16)) + ((uint64_t)n << 32);
  __syncthreads();
  uint64_t count = 0;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) count += counts[w];
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)count);
  n = __builtin_amdgcn_readfirstlane((uint32_t)(count >> 32));
  const int rank = lo >> 16, start = lo & 0xffff, slabs = band_slabs<BF16>(F, band);
  if (!sums_some<GROUPS>(n, rank, slabs)) return;

  const int words = total ? (V + 31) >> 5 : (own >> 5) + 1;
  for (int w = tid; w < words; w += THREADS) bitmap[w] = 0;
  uint64_t same[CHUNKS];
#pragma unroll
  for (int c = 0; c < CHUNKS; ++c) {
    same[c] = __ballot(kv[c] == own);
    if (lane == 0) same_s[c * WAVES + wave] = same[c];
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < CHUNKS; ++c) {
    const int id = kv[c];
    // (a look first: a frequent id would queue all its lanes at one word)
    if ((total ? id != 0x7fffffff : id < own) && !(bitmap[id >> 5] >> (id & 31) & 1u)) atomicOr(&bitmap[id >> 5], 1u << (id & 31));
    if (same[c] >> lane & 1ull) {
      int before = __popcll(same[c] & ((1ull << lane) - 1ull));
      for (int x = 0; x < c * WAVES + wave; ++x) before += __popcll(same_s[x]);
      rows[before] = tid + THREADS * c;
    }
  }
  __syncthreads();
  int set = 0;                                   // distinct ids below the own one, and all << 16
  for (int w = tid; w < words; w += THREADS) {
    const uint32_t bits = bitmap[w], low = w < own >> 5 ? ~0u : w == own >> 5 ? (1u << (own & 31)) - 1u : 0u;
    set += __popc(bits & low) | __popc(bits) << 16;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) set += __shfl_xor(set, o);
  if (lane == 0) set_s[wave] = set;
  __syncthreads();
  set = 0;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) set += set_s[w];
  const int j = __builtin_amdgcn_readfirstlane(set & 0xffff);
  sum_run<BF16, GROUPS>(dU, rows, n, rank, slabs, blockIdx.y * band, F, dE_rows + (int64_t)j * F, red);
  if (rank > 0 || blockIdx.y > 0) return;
  for (int k = tid; k < n; k += THREADS) {
    sorted_ids[start + k] = own;
    perm[start + k] = rows[k];
    seg_of[start + k] = j;
  }
  if (tid == 0) {
    uniq_ids[j] = own;
    seg_offsets[j] = start;
    if (total) { seg_offsets[set >> 16] = T; *n_uniq = set >> 16; }
  }
}

int bits_for(int V) {
  int b = 1;
  while (b < 31 && (1ll << b) < (long long)V) ++b;
  return b;
}

}  // namespace

int64_t stem_seg_chunks(int64_t max_tokens) { return (max_tokens + SEG_ROWS - 1) / SEG_ROWS; }
int64_t stem_sort_count_entries(int64_t max_tokens) {
  const int64_t tiles = (max_tokens + SORT_TILE - 1) / SORT_TILE;
  return tiles * SORT_WAVES * RADIX;
}

// One launch up to 16384 ids, of workgroups that count ranks up to 2048 and take a bucket of the vocabulary each beyond, while the
// vocabulary's bitmap is at most 32 KB (2^18 ids); beyond that vocabulary, or where buffers of the call lie over each other (those
// workgroups read the ids and store all outputs at the same time), one workgroup up to 4096 ids (8 us up to 1024, 14 us beyond, where three
// launches take 22 in a graph).  Then runs of
// 1024, while their number is one group of the merge's searches, and runs of 4096, us in a graph: 6000 ids 22 / 29, 16384
// ids 25 / 32 (one workgroup 43, the digit passes below 140), 32768 ids 36 / 34, 65536 ids 58 / 38 (digit passes 182).
// The digit passes are left to ids or batches that the packed keys or the unique kernel's quadratic reads do not suit
// (262144 ids: 126 us against 640).
// The rule by size for calls that neither ranks nor buckets sort.
int stem_route_sort(int64_t T, int V) {
  const int vbits = bits_for(V);
  if (T <= 4096 && vbits + bits_for((int)T) <= 32) return T <= 1024 ? SORT_ONE_1024 : SORT_ONE_4096;
  const bool short_runs = T <= MERGE_WAYS * 1024;
  if (T <= 262144 && vbits + (short_runs ? 10 : 12) <= 32) return short_runs ? SORT_RUNS_1024 : SORT_RUNS_4096;
  return SORT_DIGITS;
}

// Whether no two buffers of a sort overlap: workgroups that read the ids store all outputs at the same time.
static bool sort_apart(int64_t T, int V, const int32_t* ids, const int32_t* sorted_ids, const int32_t* perm, const int32_t* uniq_ids,
                       const int32_t* seg_offsets, const int32_t* n_uniq, const int32_t* seg_of) {
  const int64_t cap = std::min<int64_t>(T, V);
  const struct { const int32_t* at; int64_t n; } buf[] = {{ids, T}, {sorted_ids, T}, {perm, T}, {uniq_ids, cap}, {seg_offsets, cap + 1}, {n_uniq, 1}, {seg_of, T}};
  for (const auto& p : buf)
    for (const auto* q = buf; q < &p; ++q)
      if (reinterpret_cast<uintptr_t>(p.at) < reinterpret_cast<uintptr_t>(q->at + q->n) &&
          reinterpret_cast<uintptr_t>(q->at) < reinterpret_cast<uintptr_t>(p.at + p.n))
        return false;
  return true;
}

int stem_route_sort_ranks(int64_t T, int V, const int32_t* ids, const int32_t* sorted_ids, const int32_t* perm, const int32_t* uniq_ids,
                          const int32_t* seg_offsets, const int32_t* n_uniq, const int32_t* seg_of) {
  return T <= RANK_MAX && V <= RANK_WORDS * 32 && sort_apart(T, V, ids, sorted_ids, perm, uniq_ids, seg_offsets, n_uniq, seg_of);
}

int stem_route_sort_buckets(int64_t T, int V, const int32_t* ids, const int32_t* sorted_ids, const int32_t* perm, const int32_t* uniq_ids,
                            const int32_t* seg_offsets, const int32_t* n_uniq, const int32_t* seg_of) {
  return T > BUCKET_MIN && T <= BUCKET_MAX && V <= 256 * BUCKET_IDS && sort_apart(T, V, ids, sorted_ids, perm, uniq_ids, seg_offsets, n_uniq, seg_of);
}

hipError_t stem_sort_unique(stem_ctx* ctx, const EmbedScratch& ws, const int32_t* ids, int64_t T, int V,
                            int32_t* sorted_ids, int32_t* perm, int32_t* uniq_ids, int32_t* seg_offsets,
                            int32_t* n_uniq, hipStream_t s) {
  const int passes = (bits_for(V) + RADIX_BITS - 1) / RADIX_BITS;
  const int route = stem_route_sort(T, V);
  const int pos_bits = bits_for((int)std::min<int64_t>(T, 1 << 30));
  if (stem_route_sort_buckets(T, V, ids, sorted_ids, perm, uniq_ids, seg_offsets, n_uniq, ws.seg_of)) {
    ProfScope ps(ctx, K_SORT_FUSED, s);
    const int R = std::max(32, ((V + 255) / 256 + 31) / 32 * 32), buckets = (V + R - 1) / R;
    auto* const kernel = T <= 4096 ? sort_buckets_kernel<4> : T <= 8192 ? sort_buckets_kernel<8> : sort_buckets_kernel<16>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)buckets), dim3(1024), 0, s, ids, (int)T, V, R, bits_for(R), sorted_ids, perm, uniq_ids,
                       seg_offsets, n_uniq, ws.seg_of, ws.flag);
    return hipGetLastError();
  }
  if (stem_route_sort_ranks(T, V, ids, sorted_ids, perm, uniq_ids, seg_offsets, n_uniq, ws.seg_of)) {
    ProfScope ps(ctx, K_SORT_FUSED, s);
    auto* const kernel = T <= 1024 ? sort_ranks_kernel<1, 8> : sort_ranks_kernel<2, 8>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)((T + 7) / 8)), dim3(1024), 0, s, ids, (int)T, V, pos_bits, sorted_ids, perm,
                       uniq_ids, seg_offsets, n_uniq, ws.seg_of, ws.flag);
    return hipGetLastError();
  }
  if (route == SORT_ONE_1024 || route == SORT_ONE_4096) {
    ProfScope ps(ctx, K_SORT_FUSED, s);
    if (route == SORT_ONE_1024)
      hipLaunchKernelGGL((sort_lds_kernel<1, false>), dim3(1), dim3(1024), 0, s, ids, (int)T, V, pos_bits, passes,
                         sorted_ids, perm, uniq_ids, seg_offsets, n_uniq, ws.seg_of, ws.flag);
    else
      hipLaunchKernelGGL((sort_lds_kernel<4, false>), dim3(1), dim3(1024), 0, s, ids, (int)T, V, pos_bits, passes,
                         sorted_ids, perm, uniq_ids, seg_offsets, n_uniq, ws.seg_of, ws.flag);
    return hipGetLastError();
  }
  if (route == SORT_RUNS_1024 || route == SORT_RUNS_4096) {
    const int items = route == SORT_RUNS_4096 ? 4 : 1, run_bits = items == 1 ? 10 : 12;
    const int R = items * 1024, runs = (int)((T + R - 1) / R);
    {
      ProfScope ps(ctx, K_SORT_FUSED, s);
      if (items == 1)
        hipLaunchKernelGGL((sort_lds_kernel<1, true>), dim3(runs), dim3(1024), 0, s, ids, (int)T, V, run_bits, passes,
                           ws.sort_keys[0], ws.sort_vals[0], nullptr, nullptr, nullptr, nullptr, ws.flag);
      else
        hipLaunchKernelGGL((sort_lds_kernel<4, true>), dim3(runs), dim3(1024), 0, s, ids, (int)T, V, run_bits, passes,
                           ws.sort_keys[0], ws.sort_vals[0], nullptr, nullptr, nullptr, nullptr, ws.flag);
    }
    {
      ProfScope ps(ctx, K_SORT_MERGE, s);
      hipLaunchKernelGGL(merge_runs_kernel, dim3((unsigned)((T + 255) / 256)), dim3(256), 0, s, ws.sort_keys[0],
                         ws.sort_vals[0], (int)T, R, sorted_ids, perm);
    }
    ProfScope ps(ctx, K_UNIQUE, s);
    hipLaunchKernelGGL(unique_blocks_kernel, dim3((unsigned)((T + 1023) / 1024)), dim3(1024), 0, s, sorted_ids, (int)T,
                       uniq_ids, seg_offsets, n_uniq, ws.seg_of);
    return hipGetLastError();
  }
  const int tiles = (int)((T + SORT_TILE - 1) / SORT_TILE);
  const int nW = tiles * SORT_WAVES;
  const int32_t* src_k = ids;
  const int32_t* src_v = nullptr;
  for (int p = 0; p < passes; ++p) {
    int32_t* dst_k = (p == passes - 1) ? sorted_ids : ws.sort_keys[p & 1];
    int32_t* dst_v = (p == passes - 1) ? perm : ws.sort_vals[p & 1];
    const int shift = p * RADIX_BITS;
    {
      ProfScope ps(ctx, K_SORT_COUNT, s);
      hipLaunchKernelGGL(sort_count_kernel, dim3(tiles), dim3(1024), 0, s, src_k, T, V, shift, p == 0, nW,
                         ws.sort_counts, ws.flag);
    }
    {
      ProfScope ps(ctx, K_SORT_SCAN, s);
      hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(1024), 0, s, ws.sort_counts, nW * RADIX);
    }
    {
      ProfScope ps(ctx, K_SORT_SCATTER, s);
      hipLaunchKernelGGL(sort_scatter_kernel, dim3(tiles), dim3(1024), 0, s, src_k, src_v, T, V, shift, p == 0,
                         nW, ws.sort_counts, dst_k, dst_v, ws.flag);
    }
    src_k = dst_k;
    src_v = dst_v;
  }
  {
    ProfScope ps(ctx, K_UNIQUE, s);
    hipLaunchKernelGGL(unique_kernel, dim3(1), dim3(1024), 0, s, sorted_ids, T, uniq_ids, seg_offsets, n_uniq,
                       ws.seg_of);
  }
  return hipGetLastError();
}

// Where one launch sums whole runs, and of how many teams of four wavefronts its workgroups are.
// Up to 2048 tokens (the looks at all ids are quadratic) and 8192 workgroups, most of which end at once.  Two teams while the tokens alone
// don't fill the chip and a row has slabs for them, and up to 256 tokens two workgroups for a row of 16 slabs: us, one team / two / two
// and bands of 8 slabs: bf16, 8192 columns, 128 tokens 9.4 / 6.9 / 5.6, 256 9.9 / 7.3 / 7.0, 512 9.3 / 7.5 / 10.0; fp32 1024 x 2048 7.5 / 8.6.
static int run_slabs(int is_bf16, int F) { return (F + (is_bf16 ? 511 : 255)) / (is_bf16 ? 512 : 256); }
static bool runs_wide(int64_t T, int slabs) { return T <= 512 && slabs > 4; }
static int run_band(int64_t T, int slabs) { return T <= 256 && slabs > 4 ? 8 : MAX_BAND; }
static int run_bands(int64_t T, int slabs) { return (slabs + run_band(T, slabs) - 1) / run_band(T, slabs); }
static bool runs_fit(int is_bf16, int64_t T, int F) { return T <= SMALL_MAX && T * run_bands(T, run_slabs(is_bf16, F)) <= 8192; }

int stem_route_sort_sum(int is_bf16, int64_t T, int V, int F, const int32_t* ids, const void* dU, const int32_t* sorted_ids,
                        const int32_t* perm, const int32_t* uniq_ids, const int32_t* seg_offsets, const int32_t* n_uniq,
                        const int32_t* seg_of, const float* dE_rows) {
  if (!dU || !runs_fit(is_bf16, T, F) || V > SMALL_WORDS * 32 ||
      !stem_route_sort_ranks(T, V, ids, sorted_ids, perm, uniq_ids, seg_offsets, n_uniq, seg_of))
    return 0;
  const int64_t cap = std::min<int64_t>(T, V);
  const struct { const void* at; int64_t n; } buf[] = {{dU, T * F * (is_bf16 ? 2 : 4)}, {dE_rows, cap * F * 4}, {ids, T * 4},
      {sorted_ids, T * 4}, {perm, T * 4}, {uniq_ids, cap * 4}, {seg_offsets, cap * 4 + 4}, {n_uniq, 4}, {seg_of, T * 4}};
  for (const auto& p : buf)
    for (const auto* q = buf; q < buf + 2 && q < &p; ++q) {
      const uintptr_t a = reinterpret_cast<uintptr_t>(p.at), b = reinterpret_cast<uintptr_t>(q->at);
      if (a < b + q->n && b < a + p.n) return 0;
    }
  return 1;
}

hipError_t stem_table_grad(stem_ctx* ctx, const EmbedScratch& ws, int is_bf16, const int32_t* ids, const void* dU, int64_t T, int V, int F,
                           int32_t* sorted_ids, int32_t* perm, int32_t* uniq_ids, int32_t* seg_offsets, int32_t* n_uniq, float* dE_rows,
                           hipStream_t s) {
  if (stem_route_sort_sum(is_bf16, T, V, F, ids, dU, sorted_ids, perm, uniq_ids, seg_offsets, n_uniq, ws.seg_of, dE_rows)) {
    ProfScope ps(ctx, K_SEG_REDUCE, s);
    const int slabs = run_slabs(is_bf16, F);
    const bool wide = runs_wide(T, slabs);
    auto* const kernel = T > 1024 ? (is_bf16 ? sort_sum_kernel<true, 1, 2048> : sort_sum_kernel<false, 1, 2048>)
                         : wide   ? (is_bf16 ? sort_sum_kernel<true, 2, 1024> : sort_sum_kernel<false, 2, 1024>)
                                  : (is_bf16 ? sort_sum_kernel<true, 1, 1024> : sort_sum_kernel<false, 1, 1024>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)T, (unsigned)run_bands(T, slabs)), dim3(wide ? 512 : 256), 0, s, ids, (int)T, V, dU, F,
                       run_band(T, slabs), sorted_ids, perm, uniq_ids, seg_offsets, n_uniq, ws.seg_of, dE_rows, ws.flag);
    return hipGetLastError();
  }
  const hipError_t e = stem_sort_unique(ctx, ws, ids, T, V, sorted_ids, perm, uniq_ids, seg_offsets, n_uniq, s);
  return e != hipSuccess || !dU ? e : stem_seg_reduce(ctx, ws, is_bf16, dU, perm, seg_offsets, T, F, dE_rows, s);
}

hipError_t stem_seg_reduce(stem_ctx* ctx, const EmbedScratch& ws, int is_bf16, const void* dU, const int32_t* perm,
                           const int32_t* seg_offsets, int64_t T, int F, float* dE_rows, hipStream_t s) {
  const int chunks = (int)((T + SEG_ROWS - 1) / SEG_ROWS);
  const int cols = is_bf16 ? 8 : 4;
  if (runs_fit(is_bf16, T, F)) {
    ProfScope ps(ctx, K_SEG_REDUCE, s);
    const int slabs = run_slabs(is_bf16, F);
    const bool wide = runs_wide(T, slabs);
    auto* const kernel = wide ? (is_bf16 ? seg_runs_kernel<true, 2> : seg_runs_kernel<false, 2>)
                              : (is_bf16 ? seg_runs_kernel<true, 1> : seg_runs_kernel<false, 1>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)T, (unsigned)run_bands(T, slabs)), dim3(wide ? 512 : 256), 0, s, dU, perm, ws.seg_of,
                       seg_offsets, F, run_band(T, slabs), dE_rows);
    return hipGetLastError();
  }
  const int slabs = (F + 256 * cols - 1) / (256 * cols);
  {
    ProfScope ps(ctx, K_SEG_REDUCE, s);
    if (is_bf16)
      hipLaunchKernelGGL(seg_reduce_kernel<true>, dim3(slabs, chunks), dim3(256), 0, s, dU, perm, ws.seg_of, T, F,
                         dE_rows, ws.seg_part);
    else
      hipLaunchKernelGGL(seg_reduce_kernel<false>, dim3(slabs, chunks), dim3(256), 0, s, dU, perm, ws.seg_of, T,
                         F, dE_rows, ws.seg_part);
  }
  {
    ProfScope ps(ctx, K_SEG_COMBINE, s);
    if (is_bf16)
      hipLaunchKernelGGL(seg_combine_kernel<8>, dim3(chunks, (F + 511) / 512), dim3(256), 0, s, ws.seg_of, seg_offsets, T,
                         F, dE_rows, ws.seg_part);
    else
      hipLaunchKernelGGL(seg_combine_kernel<4>, dim3(chunks, (F + 255) / 256), dim3(256), 0, s, ws.seg_of, seg_offsets, T,
                         F, dE_rows, ws.seg_part);
  }
  return hipGetLastError();
}
