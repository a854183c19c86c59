// bf16 MFMA GEMMs of the STEM layer (gate, down, and the four backward products)
// for gfx950, with the layer's element-wise work fused into the epilogues.
//
// One kernel template computes  C[m,n] = sum_k Aop[m,k] * Bop[n,k]  on one output tile per
// workgroup: 256x256 for products with enough of them to fill the chip, else 256x128, 192x128 or 128x128
// (see Tiling; choose_plan decides, and may also cut K into slices).  The 256x256 tile: 4 wavefronts,
// each a 128x128 quadrant held as 4x4 accumulators of v_mfma_f32_32x32x16_bf16, K stepped by 64
// through a ring of five 32 KB LDS slots (one operand tile each), so that every global request is made
// more than a whole K tile before its data is needed.
//
// Operands.  "KC" = stored [rows,K] with K contiguous, "MC" = stored [K,rows] with rows
// contiguous.  Tiles of both kinds go global -> LDS directly (buffer_load ... lds, 16 bytes per
// lane, whole 128-byte lines; half lines were measured to halve the L1 rate) and keep the
// orientation they have in memory; what differs is the fragment read.  A KC tile gives an MFMA
// fragment (8 consecutive k of one row) as one 16-byte LDS read; an MC tile gives it as two
// ds_read_b64_tr_b16, the LDS read of gfx950 that transposes 16-bit values across 16 lanes.  So
// no operand is ever transposed in memory or in registers: the backward products read the
// weights, the activations and their gradients exactly as the forward pass left them.  (An
// earlier version staged MC tiles through registers with byte permutes and needed the other
// operand K-contiguous, i.e. four transposing kernels per backward pass; its weight-gradient
// loops ran at 2800-3060 clocks per K tile against 2050-2300 for this one.)  All loads are
// buffer loads: out-of-range rows / k read as zero, so ragged edges need no branches.
//
// LDS layout of a KC tile: row r (an m or n index within the tile) owns 128 bytes = 8 chunks of
// 8 bf16; chunk c of row r sits at chunk slot (c ^ (r >> 1) ^ (((r >> 3) & 3) << 1)) & 7.  With
// the first term a ds_read_b128 of one chunk column over 16 consecutive rows touches all 64
// banks once (measured per instruction with four wavefronts issuing: 16 clocks, conflict-free).
// The layout of an MC tile is described at its loader.
//
// Schedule of the 256x256 tile.  One iteration = one K tile = 4 k-steps of 16 MFMAs.  Fragments are double
// buffered in registers: while the MFMAs of k-step s run, the 8 fragment reads of step
// s+1 are issued between them.  The loads of later tiles are spread over the k-steps
// (a vector-memory instruction blocks the issuing wavefront for tens of cycles, during
// which its MFMA queue drains, so they are never issued back to back).  The single
// barrier per iteration sits before the last k-step, so that step overlaps the first
// fragment reads of the next tile, and the wait before it leaves the youngest requests
// in flight.  The loop is unrolled over the slot rotation (5 K tiles) so that every
// LDS address is a loop-invariant register plus an immediate.
//
// Epilogue.  The MFMA is issued with the N-side fragment as its row operand, so a lane
// holds, for one m, groups of 4 consecutive n.  Each wavefront stages its accumulators
// through LDS (fp32, 32 rows at a time) and reads them back row-contiguous: 16 lanes
// cover 128 consecutive n of one row, so the outputs, the gathered table row and the
// saved activations are all accessed as 16-byte pieces of whole 128-byte lines.
#include "stem_internal.h"

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef __amdgpu_buffer_rsrc_t rsrc_t;

namespace {

constexpr int BK = 64;
constexpr uint32_t OOB = 0x80000000u;  // a buffer offset beyond any operand: reads as zero

__device__ __forceinline__ uint32_t lds_addr(const char* p) {   // p points into LDS
  return (uint32_t)(uintptr_t)(lds_ptr_t)const_cast<char*>(p);
}
// chunk slot swizzle of a row of a K-contiguous tile (only bits 1..4 of the row: the same for rows 32
// apart, so the fragments of a wavefront's four 32-row blocks sit at one address plus immediates)
__device__ __forceinline__ int lds_swz(int row) { return ((row >> 1) ^ (((row >> 3) & 3) << 1)) & 7; }

// A buffer resource that moves along the operand: base advances, the record count shrinks, to zero at the operand's end
// and not below: the loaders request up to three K tiles beyond it, and three K tiles of an operand whose rows are
// millions of elements long are more than an int holds.
// The descriptor is rebuilt once per K tile (a handful of scalar instructions), not per load.
struct Window {
  const char* base;
  int left;  // bytes from base to the end of the operand (operands stay below 2 GiB), zero past it
  rsrc_t r;
  __device__ __forceinline__ void set(const void* p, int64_t bytes) {
    base = reinterpret_cast<const char*>(p);
    left = bytes < 0 ? 0 : (int)bytes;
    rebuild();
  }
  __device__ __forceinline__ void rebuild() { r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0, left, 0x00020000); }
  __device__ __forceinline__ rsrc_t rsrc() const { return r; }
  // the same descriptor as four words (base, stride 0, byte count, raw-buffer flags), for loads issued as assembly
  __device__ __forceinline__ u32x4_t words() const {
    const uint64_t b = reinterpret_cast<uint64_t>(base);
    return u32x4_t{(uint32_t)b, (uint32_t)(b >> 32) & 0xffffu, (uint32_t)left, 0x00020000u};
  }
  __device__ __forceinline__ void advance(int bytes) {   // bytes: a K tile, less than 2^30
    base += bytes;
    const int l = left - bytes;
    left = l < 0 ? 0 : l;
    rebuild();
  }
};

// One direct-to-LDS load of 16 bytes per lane, written as assembly.  The compiler orders every
// transposing LDS read (ds_read_b64_tr_b16) after ALL outstanding direct-to-LDS loads it knows of
// (a wait for vmcnt(0) in front of each), which would drain the ring in every k-step; products
// with a rows-contiguous operand therefore issue their loads where the compiler does not see
// them.  Nothing returns to a register, and the kernel's own waits (vmcnt before each barrier) are
// what orders these loads against the reads, as they do for the compiler-made ones.  M0 (the LDS
// destination) is written inside the statement; the compiler never keeps a value of its own in M0
// across other code (it sets it directly in front of each instruction that reads it).
__device__ __forceinline__ void lds_dma_16(u32x4_t rs, uint32_t lds_dst, uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds_dst), "v"(off), "s"(rs) : "memory");
}

// the same load through the compiler (a function of its own: inside a template the host pass drops the builtin's caller)
__device__ __forceinline__ void lds_dma_16_known(rsrc_t rs, char* lds_dst, uint32_t off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)lds_dst, 16, off, 0, 0, 0);
}

// ---- KC operand: global -> LDS direct -----------------------------------------------
// Wavefront w loads row groups g = w*8 + i (8 rows each); lane -> row g*8 + (lane >> 3),
// chunk slot lane & 7; the lane fetches the chunk that belongs in its slot.
template <int EDGE, int WAVES>
struct LoaderKC {
  static constexpr int LOADS = EDGE / 8 / WAVES;   // per wavefront and tile
  uint32_t off[LOADS];
  Window win;
  // `skip`: elements by which p already points past the operand's first element (a K slice)
  __device__ __forceinline__ void init(const bf16_t* p, int ld, int rows, int row0, int wave, int lane, int skip) {
    win.set(p, ((int64_t)rows * ld - skip) * 2);
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int row = (wave * LOADS + i) * 8 + (lane >> 3);
      const int c = (lane & 7) ^ lds_swz(row);
      off[i] = (row0 + row) < rows ? (uint32_t)(((int64_t)(row0 + row) * ld + c * 8) * 2) : OOB;
    }
  }
  // load i of the tile the window points at, into `tile` (LDS, wave-uniform)
  __device__ __forceinline__ void issue(int i, char* tile, int wave) const {
    lds_dma_16_known(win.rsrc(), tile + (wave * LOADS + i) * 1024, off[i]);
  }
  __device__ __forceinline__ void issue_opaque(int i, char* tile, int wave) const {
    lds_dma_16(win.words(), lds_addr(tile + (wave * LOADS + i) * 1024), off[i]);
  }
  __device__ __forceinline__ void next_tile() { win.advance(BK * 2); }
};

// ---- MC operand: global -> LDS as stored, transposed by the fragment reads ----------------
// The 64 x 256 tile keeps the operand's own orientation in LDS: K row k owns 512 bytes = 32 chunks
// of 8 rows-of-the-product (m or n), chunk c at chunk slot c ^ ((k & 3) << 2).  A wavefront's load
// instruction fills 1 KB = two K rows; the lane fetches the chunk that belongs in its slot, so 32
// lanes read one 512-byte stretch of a global row.  ds_read_b64_tr_b16 then delivers MFMA fragments:
// within 16 lanes, lane 4a + b supplies the address of 4 consecutive 16-bit values of "row" a, piece
// b, and lane j receives the j-th value of rows 0..3 (checked on the device with an index pattern).
// With a = k and b = 4-column piece, lane j ends up with 4 consecutive k of column j: half a
// fragment.  The slot swizzle puts the four K rows that 16 lanes read in different 64-byte bank
// groups, so 32 lanes (one LDS pass of a 64-bit read) touch all 64 banks once.
template <int EDGE, int WAVES>
struct LoaderMC {
  static constexpr int LOADS = EDGE / 8 / WAVES;
  static constexpr int CHUNKS = EDGE / 8;          // 16-byte chunks of a K row
  static constexpr int ROW_BYTES = CHUNKS * 16;
  uint32_t off[LOADS];
  uint32_t tile_bytes;   // one K tile further along the operand
  Window win;
  __device__ __forceinline__ void init(const bf16_t* p, int ld, int rows, int K, int row0, int wave, int lane) {
    win.set(p, (int64_t)K * ld * 2);
    tile_bytes = (uint32_t)ld * (BK * 2);
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int k = (wave * LOADS + i) * (64 / CHUNKS) + lane / CHUNKS;
      const int c = (lane & (CHUNKS - 1)) ^ ((k & 3) << 2);
      off[i] = (row0 + c * 8) < rows ? (uint32_t)(((int64_t)k * ld + row0 + c * 8) * 2) : OOB;
    }
  }
  __device__ __forceinline__ void issue(int i, char* tile, int wave) const {
    lds_dma_16(win.words(), lds_addr(tile + (wave * LOADS + i) * 1024), off[i]);
  }
  __device__ __forceinline__ void next_tile() { win.advance((int)tile_bytes); }
  // Byte offset within a tile of this lane's address for the first half (k + 0..3) of fragment i
  // (rows base + i*32 .. +31 of the product tile) of k-step 0; the second half is 4 K rows on, k-step
  // s another 16 s.  Lane = 16 g + 4 a + b: K row 8 (g >> 1) + a, rows 16 (g & 1) + 4 b .. + 3.
  static __device__ __forceinline__ uint32_t frag_off(int base, int i, int lane) {
    const int g = lane >> 4, a = (lane >> 2) & 3, b = lane & 3;
    const int c = base / 8 + i * 4 + 2 * (g & 1) + (b >> 1);
    return (uint32_t)((8 * (g >> 1) + a) * ROW_BYTES + ((c ^ (a << 2)) << 4) + 8 * (b & 1));
  }
};
typedef __attribute__((ext_vector_type(4))) short s16x4_t;
typedef __attribute__((ext_vector_type(8))) short s16x8_t;
// one MFMA fragment (8 consecutive k of this lane's row) from a tile in the layout above
template <int ROW_BYTES>
__device__ __forceinline__ bf16x8_t lds_read_frag_tr(const char* p) {
  typedef __attribute__((address_space(3))) s16x4_t* lds_s16x4_ptr;
  const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(lds_ptr_t) const_cast<char*>(p));
  const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(lds_ptr_t) const_cast<char*>(p + 4 * ROW_BYTES));
  return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// ---- epilogue math ------------------------------------------------------------------
__device__ __forceinline__ float sigmoidf_fast(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }
__device__ __forceinline__ uint4 pack8(const float (&f)[8]) {
  bf16x8_t v;
#pragma unroll
  for (int q = 0; q < 8; ++q) v[q] = (__bf16)f[q];
  return __builtin_bit_cast(uint4, v);
}
__device__ __forceinline__ void unpack8(uint4 u, float (&f)[8]) {
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    f[2 * q] = __uint_as_float(w[q] << 16);
    f[2 * q + 1] = __uint_as_float(w[q] & 0xffff0000u);
  }
}

// Workgroup -> output tile.  Consecutive workgroup ids go round-robin over the 8 XCDs,
// each with its own L2; giving every XCD one contiguous run of tiles, walked in bands of
// GM tile-rows (down the rows of a band first), keeps the operand panels an XCD's workgroups
// share in that XCD's L2.  GM = 4: the 32 workgroups an XCD runs at a time cover 4 tile-rows
// x 8 tile-columns, i.e. 4 panels of the M-side operand (activations or their gradients, rows
// no other XCD reads) and 8 of the N-side one (mostly weights, which all XCDs read and the
// memory-side cache therefore holds).  With GM = 8 (8 + 4 panels, the same count) every product
// was 1-3 % slower.  The dH product takes GM = 7, which divides neither the 32 tiles an XCD runs
// at a time nor its run: the XCDs then sit at different rows and columns of their bands, and
// their epilogues (each reads a G tile and writes two tiles) meet less often: 0.565 ms with
// 8, 0.545 with 4 or 6, 0.537 with 3 or 5, 0.532 with 7, 0.545-0.55 with 9, 11, 13
// (d_model 2048, d_ff 8192, 16384 tokens).
__host__ __device__ __forceinline__ int xcd_major(int b, int nb) {
  const int q = nb >> 3, r = nb & 7;
  const int xcd = b & 7, idx = b >> 3;
  return xcd * q + (xcd < r ? xcd : r) + idx;
}
__host__ __device__ __forceinline__ void tile_at(int gm, int L, int ntm, int ntn, int& tm, int& tn) {
  const int per_group = gm * ntn;
  const int group = L / per_group;
  const int first = group * gm;
  const int gsize = (ntm - first) < gm ? (ntm - first) : gm;
  const int in = L - group * per_group;
  tm = first + in % gsize;
  tn = in / gsize;
}
// Workgroup -> K slice, product and place in the product's bands, for launches of several products (n_more beyond the first, of
// which tiles0 and tiles1 are the tiles of the first two) or K slices: the slices follow each other in the XCDs' runs of tiles, so
// that an XCD works on one or two of them (1024 x 4096 weight gradient, 16384 tokens, 4 slices: 123.5 us with every slice on
// every XCD, 122.2), and in each slice the products.
struct Place { int slice, product, in; };
__host__ __device__ __forceinline__ Place place_of(int b, int nb, int ksplit, int n_more, int tiles0, int tiles1) {
  const int all = nb / ksplit, L = xcd_major(b, nb);
  Place q = {L / all, 0, L % all};
  if (n_more > 0 && q.in >= tiles0) {
    q.product = 1;
    q.in -= tiles0;
    if (n_more > 1 && q.in >= tiles1) {
      q.product = 2;
      q.in -= tiles1;
    }
  }
  return q;
}

// A tiling: a wavefront holds MI x NJ accumulators of 32 x 32, WM x WN wavefronts multiply, and the operand
// tiles pass through the five-slot ring (STAGES = 0) or through STAGES whole K tiles of LDS that LW further
// wavefronts do nothing but fill.
//
// Tile256 (160 KB of LDS, 256 accumulator registers) moves the fewest operand bytes per FLOP, 32 per clock and CU
// at full MFMA rate, and is the one for products that fill the chip with 256 x 256 tiles.  Below that a smaller
// tile keeps all CUs busy.  The smaller ones need 48 and 64 bytes per clock and CU and are bound by operand loads
// (with MFMAs and fragment reads taken out they take as long), so what counts for them is the bytes in flight: a
// loads-only walk of 128 x 128 tiles reaches 63 GB/s per CU with one K tile in flight and 105 with two; three stages
// keep two in flight, and five bring nothing more.  The separate load wavefronts keep the multiplying ones from
// stalling on load issue (2048 x 8192 down product, 256 tokens: 47.5 us without, 43.3 with; 256 x 128 tiles, 4096
// tokens: 116.6 and 113.9).  Tile256 has no registers left for them.  Two workgroups of 128 x 128 tiles per CU on
// an 80 KB ring were 1.3 x slower where one per CU is enough (57 us against 43) and equal elsewhere.
template <int MI_, int NJ_, int WM_, int WN_, int STAGES_, int LW_>
struct Tiling {
  static constexpr int MI = MI_, NJ = NJ_, WM = WM_, WN = WN_, STAGES = STAGES_, LW = LW_;
  static constexpr int TM = 32 * MI * WM, TN = 32 * NJ * WN, WAVES = WM * WN;
  static constexpr int A_BYTES = TM * BK * 2, B_BYTES = TN * BK * 2;   // one operand tile in LDS
  static constexpr int LDS_BYTES = STAGES == 0 ? 5 * A_BYTES : STAGES * (A_BYTES + B_BYTES);
};
typedef Tiling<4, 4, 2, 2, 0, 0> Tile256;
typedef Tiling<4, 2, 2, 2, 3, 4> Tile256x128;
typedef Tiling<2, 2, 2, 2, 3, 4> Tile128;
// 700 tokens of an 8192-wide gate product are 96 tiles of 256x256, 192 of 256x128, 384 of 128x128 and 256 of these.  A whole product
// keeps a compute unit at about 60 GB/s once all 256 load (40 KB a K tile in 0.69 us, the model's `full`; 0.33 us, 124 GB/s, with a
// few), so in one full round the bytes of a tile count: 40 KB a K tile here against 48 on 192 units, or 32 in one and a half rounds
// (gate 34.1 -> 30.7 us; down product in four slices 39.3 -> 33.4).
typedef Tiling<3, 2, 2, 2, 3, 4> Tile192x128;

template <class C, int LA, int LB, int EPI>
__global__ __launch_bounds__((C::WAVES + C::LW) * 64) void gemm_bf16_kernel(GemmArgs p) {
  constexpr int MI = C::MI, NJ = C::NJ;
  constexpr int WSM = 32 * MI, WSN = 32 * NJ;  // a wavefront's piece of the tile
  constexpr int TILE_BYTES = C::A_BYTES;       // ring: one slot (both operands alike)
  constexpr int LOADERS = C::LW ? C::LW : C::WAVES;   // wavefronts that issue loads
  typedef LoaderKC<C::TM, LOADERS> LoadAKC;
  typedef LoaderMC<C::TM, LOADERS> LoadAMC;
  typedef LoaderKC<C::TN, LOADERS> LoadBKC;
  typedef LoaderMC<C::TN, LOADERS> LoadBMC;
  constexpr int LOADS_A = LoadAKC::LOADS, LOADS_B = LoadBKC::LOADS;   // loads per wavefront and tile
  __shared__ __attribute__((aligned(16))) char smem[C::LDS_BYTES];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave_id = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool load_wave = C::LW && wave_id >= C::WAVES;
  const int wave = load_wave ? wave_id - C::WAVES : wave_id;
  const int wm = wave / C::WN, wn = wave % C::WN;
  // Gate and up product in one: half of a wavefront's columns are C's, the other half Up's, so that the tile's B rows are, 32 * NJ / 2 at
  // a time, of W_gate and of W_up in turn: what a loader brings is of one of them.  As two launches the second
  // read Up back in an epilogue under which nothing else runs, all tiles at once, and small batches paid a launch, a prologue and a
  // split product's sum more.  Forward call, us, two launches / one, additive and dense layer: 1024 x 4096, 300 tokens 36.1 / 26.2 and
  // 34.6 / 25.9, 4096 tokens 123.2 / 116.5 and 107.8 / 102.2, 16384 tokens 425 / 398 and 401 / 378; 1216 x 3328, 5000 tokens 167 / 144 and
  // 161 / 141; 2048 x 8192, 700 tokens 95.2 / 91.3 and 93.5 / 89.3, 16384 tokens 1352 / 1319 and 1308 / 1286.  The tiling is choose_plan's
  // for a product of twice the width, and the best of the four or within 3 % of it at 16 layers.
  constexpr bool DUAL = EPI == EPI_GATE_DUAL || EPI == EPI_GATE_DUALE;
  static_assert(!DUAL || LOADERS == 2 * C::WN, "a loader's B rows are one half of a wavefront's columns");
  constexpr int OUT_TN = DUAL ? C::TN / 2 : C::TN;   // columns of the output per tile
  int ntm = (p.M + C::TM - 1) / C::TM, ntn = (p.N + OUT_TN - 1) / OUT_TN;
  constexpr int BAND = (EPI == EPI_DH || EPI == EPI_DH_UP || EPI == EPI_DH_UPE) ? 7 : 4;   // see tile_at
  int tm, tn;
  Place at;
  if (EPI == EPI_F32) {
    constexpr bool SEVERAL = LA == OP_MC && LB == OP_MC;
    const int second = SEVERAL ? ((p.more[0].M + C::TM - 1) / C::TM) * ((p.more[0].N + C::TN - 1) / C::TN) : 0;
    at = place_of(blockIdx.x, gridDim.x, p.ksplit, SEVERAL ? p.n_more : 0, ntm * ntn, second);
    if (SEVERAL) {
      auto next = [&](const auto& m) __attribute__((always_inline)) {
        p.ws += (size_t)p.M * p.N;
        p.A = m.A; p.B = m.B; p.C = m.C; p.M = m.M; p.N = m.N; p.lda = m.lda; p.ldb = m.ldb;
        ntm = (p.M + C::TM - 1) / C::TM; ntn = (p.N + C::TN - 1) / C::TN;
      };
      if (at.product > 0) {
        next(p.more[0]);
        if (at.product > 1) next(p.more[1]);
      }
    }
  } else {
    at = {0, 0, xcd_major(blockIdx.x, gridDim.x)};
  }
  if (EPI == EPI_F32 && p.ksplit > 1) {
    // Split along K (few output tiles, long K): slice z of the K tiles, its product stored plainly to
    // slice z of the partial buffer; a second kernel sums the slices in order.  The slice is
    // expressed by moving the operands and shrinking K.
    const int z = at.slice;
    int zk = z, slices = p.ksplit;
    if (LA == OP_KC && p.A2) {   // two operand pairs of the same K: half of the slices each
      slices >>= 1;
      if (zk >= slices) { zk -= slices; p.A = p.A2; p.B = p.B2; }
      p.A2 = nullptr;
    }
    const int nk_all = (p.K + BK - 1) / BK;
    const int per = (nk_all + slices - 1) / slices;
    const int k0 = zk * per * BK;
    int klen = p.K - k0;
    if (klen > per * BK) klen = per * BK;
    if (klen < 0) klen = 0;
    p.A += LA == OP_KC ? (size_t)k0 : (size_t)k0 * p.lda;
    p.B += LB == OP_KC ? (size_t)k0 : (size_t)k0 * p.ldb;
    p.K = klen;
    p.kc_skip = k0;                                          // K-contiguous windows end k0 elements earlier
    p.C = p.ws + (size_t)z * p.elems;
    p.accumulate = 0;
  }
  tile_at(BAND, at.in, ntm, ntn, tm, tn);
  const int m0 = tm * C::TM, n0 = tn * OUT_TN;
  if (DUAL && (wave & 1)) p.B = p.Bup;
  // K rotation.  Workgroups on XCD x start their K loop x eighths of the way in and wrap around, so
  // the eight XCDs stream eight different stretches of the operands' rows at any moment instead of
  // the same one (measured: the down product, whose two operands have the same 16 KB row pitch, ran
  // 8 % slower without it; the other products with two direct operands are unchanged, and the
  // weight-gradient products gained nothing from the same rotation, so they do not rotate).  The sum over k is the same set of products in
  // a rotated order.  `rot` is the first K element of this workgroup's loop; 0 = no rotation.
  int rot = 0;
  if (LA == OP_KC && LB == OP_KC && !p.A2) {
    const int nk_all = (p.K + BK - 1) / BK;
    if (nk_all >= 16) rot = (int)((long)(blockIdx.x & 7) * nk_all / 8) * BK;
  }
  if (LA == OP_KC && LB == OP_KC && rot > 0) {   // expressed as two operand pairs: [rot, K) of A, B and then [0, rot)
    p.A2 = p.A; p.B2 = p.B; p.K2 = rot;
    p.A += rot; p.B += rot; p.K -= rot; p.kc_skip += rot;
  }

  f32x16_t acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  LoadAKC ka;
  LoadBKC kb_;
  LoadAMC da;
  LoadBMC db;
  if (LA == OP_KC) ka.init(p.A, p.lda, p.M, m0, wave, lane, p.kc_skip); else da.init(p.A, p.lda, p.M, p.K, m0, wave, lane);
  if (LB == OP_KC) kb_.init(p.B, p.ldb, p.N, DUAL ? n0 - ((wave + 1) >> 1) * (LOADS_B * 8) : n0, wave, lane, p.kc_skip); else db.init(p.B, p.ldb, p.N, p.K, n0, wave, lane);

  // fragments: lane -> row (lane & 31) of a 32-row block, k half (lane >> 5) of a k-step
  const int frow = lane & 31, fk = lane >> 5;

  // A second operand pair (A2, B2, K2; same layouts and leading dimensions as the first; A
  // K-contiguous) continues the sum: after the K tiles of the first pair the windows move to the second.
  const int nk1 = (p.K + BK - 1) / BK;
  const int nk = nk1 + ((LA == OP_KC && p.A2) ? (p.K2 + BK - 1) / BK : 0);
  // The gate epilogue reads one gathered table row per output row.  A few K tiles before the end
  // of the main loop each lane touches the 128-byte lines its wavefront will need, so that they
  // travel from HBM to L2 under the MFMA work instead of in a burst when all workgroups reach
  // their epilogues together.  (Measured: 0.05 ms off the gate product at d=2048, F=8192; the dH
  // product gains nothing from the same trick - its lines are evicted again before the epilogue,
  // FETCH_SIZE grows by 30 % - so it does not touch.)
  // The touching loads return asynchronously into their destination registers, so these stay
  // reserved (never reused by the compiler) until the wait that follows the main loop.
  constexpr bool TOUCH = (EPI == EPI_GATE);
  // Token ids of this wavefront's output rows (128, 96 or 64), lane l holding rows l and 64 + l, fetched here so
  // that their latency passes under the main loop.  The epilogue takes each row's id from these
  // registers by a lane permute: loading ids there would put a wait for the newest loads in front of
  // every block of table-row requests, and with it a wait for all the stores issued before them
  // (loads and stores return through one in-order counter), 3 to 4 us per block.
  constexpr bool NEED_IDS = (EPI == EPI_GATE || EPI == EPI_DH || EPI == EPI_GATE_UPE || EPI == EPI_DH_UPE || EPI == EPI_GATE_DUALE);
  int row_id[(MI + 1) / 2] = {};
  if (NEED_IDS && !load_wave) {
#pragma unroll
    for (int h = 0; h < (MI + 1) / 2; ++h) {
      const int m = m0 + wm * WSM + h * 64 + lane;
      int id = p.ids[m < p.M ? m : p.M - 1];
      if ((unsigned)id >= (unsigned)p.E_rows) {   // reported to the host, clamped so no access leaves the table
        *p.flag = 1;
        id = id < 0 ? 0 : p.E_rows - 1;
      }
      row_id[h] = id;
    }
  }
  uint32_t touched[MI] = {};
  auto touch_epilogue_inputs = [&]() {
    if (!TOUCH) return;
    const int ncol = n0 + wn * WSN;
    const int col = ncol < p.N ? ncol : 0;
#pragma unroll
    for (int h = 0; h < (MI + 1) / 2; ++h) {
      const int id = row_id[h];
      const bf16_t* e = p.E + (size_t)id * p.N + col;
      if (NJ == 2) {   // 64 columns: one line
        asm volatile("global_load_dword %0, %1, off" : "=&v"(touched[h]) : "v"(e) : "memory");
        continue;
      }
      // the second line of the row's 128 columns exists only if the matrix is that wide (d_ff may be
      // 64 modulo 128): otherwise touch the first line twice rather than the next row's memory
      const bf16_t* e2 = col + 64 < p.N ? e + 64 : e;
      asm volatile("global_load_dword %0, %2, off\n\tglobal_load_dword %1, %3, off"
                   : "=&v"(touched[(2 * h) % MI]), "=&v"(touched[(2 * h + 1) % MI]) : "v"(e), "v"(e2) : "memory");
    }
  };
  const int touch_at = nk > 8 ? ((nk - 6) & ~1) : -1;   // an even K tile index a few tiles before the end
  bf16x8_t xa[MI], xb[NJ], ya[MI], yb[NJ];
  int a_to_switch = p.A2 ? nk1 : -1, b_to_switch = a_to_switch;
  auto next_A = [&]() {
    if constexpr (LA == OP_KC) {
      if (--a_to_switch == 0) ka.win.set(p.A2, ((int64_t)p.M * p.lda - (p.kc_skip - rot)) * 2); else ka.next_tile();
    } else {
      da.next_tile();
    }
  };
  auto next_B = [&]() {
    if constexpr (LB == OP_KC) {
      if (--b_to_switch == 0) kb_.win.set(p.B2, ((int64_t)p.N * p.ldb - (p.kc_skip - rot)) * 2); else kb_.next_tile();
    } else {
      if (--b_to_switch == 0) db.win.set(p.B2, (int64_t)p.K2 * p.ldb * 2); else db.next_tile();
    }
  };
  constexpr bool OPAQUE = (LA == OP_MC || LB == OP_MC);   // see lds_dma_16
  auto issue_A = [&](int q, char* tile) {
    if constexpr (LA != OP_KC) da.issue(q, tile, wave);
    else if constexpr (OPAQUE) ka.issue_opaque(q, tile, wave);
    else ka.issue(q, tile, wave);
  };
  auto issue_B = [&](int q, char* tile) {
    if constexpr (LB != OP_KC) db.issue(q, tile, wave);
    else if constexpr (OPAQUE) kb_.issue_opaque(q, tile, wave);
    else kb_.issue(q, tile, wave);
  };
  constexpr int MCA_ROW = LoadAMC::ROW_BYTES, MCB_ROW = LoadBMC::ROW_BYTES;
  // This lane's fragment address within a tile.  x = k-step for a K-contiguous operand (whose swizzle depends on
  // it; the fragment index is an immediate), x = fragment for a rows-contiguous one (the other way round).
  auto frag_addr_A = [&](int x) -> uint32_t {
    if (LA == OP_MC) return LoadAMC::frag_off(wm * WSM, x % MI, lane);
    return (uint32_t)((wm * WSM + frow) * 128) + (uint32_t)((((x * 2 + fk) ^ lds_swz(frow)) & 7) << 4);
  };
  auto frag_addr_B = [&](int x) -> uint32_t {
    if (LB == OP_MC) return LoadBMC::frag_off(wn * WSN, x % NJ, lane);
    return (uint32_t)((wn * WSN + frow) * 128) + (uint32_t)((((x * 2 + fk) ^ lds_swz(frow)) & 7) << 4);
  };
  // fragment i of k-step ks; addr[] = frag_addr of the operand's tile
  auto frag_A = [&](const char* tile, const uint32_t(&addr)[4], int ks, int i) -> bf16x8_t {
    if constexpr (LA == OP_KC) return *reinterpret_cast<const bf16x8_t*>(tile + addr[ks] + i * 4096);
    else return lds_read_frag_tr<MCA_ROW>(tile + addr[i] + ks * 16 * MCA_ROW);
  };
  auto frag_B = [&](const char* tile, const uint32_t(&addr)[4], int ks, int i) -> bf16x8_t {
    if constexpr (LB == OP_KC) return *reinterpret_cast<const bf16x8_t*>(tile + addr[ks] + i * 4096);
    else return lds_read_frag_tr<MCB_ROW>(tile + addr[i] + ks * 16 * MCB_ROW);
  };
  auto mma = [&](int i, int j, bf16x8_t(&fa)[MI], bf16x8_t(&fb)[NJ]) {
    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
  };
  if constexpr (C::STAGES == 0) {
  // ---- main loop: ring of five 32 KB slots -----------------------------------------------------
  // Operand tiles alternate through the slots: A of K tile t in slot 2t mod 5, B in slot 2t+1 mod 5.
  // While K tile t is multiplied, A(t+1), B(t+1) are landing or landed and A(t+2) is requested
  // during the first two k-steps into the slot B(t-1) left; after the barrier that ends the reads
  // of K tile t, B(t+2) is requested into A(t)'s slot.  Every request thus has a whole K tile's
  // time (B) or more (A) before it is waited for, a request is always in flight across the
  // barrier, and the wait before the barrier leaves the youngest 8 loads pending.  With two 64 KB
  // stages the loads of a K tile were requested and drained within that tile's own time, and the
  // direct-load stream alone (no MFMA, no fragment reads) took as long as the whole kernel.
  uint32_t ra_addr[3][4], rb_addr[3][4];   // [slot pair][x]; the odd slot of a pair is an immediate away
#pragma unroll
  for (int pr = 0; pr < 3; ++pr)
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      ra_addr[pr][x] = (uint32_t)(pr * 2 * TILE_BYTES) + frag_addr_A(x);
      rb_addr[pr][x] = (uint32_t)(pr * 2 * TILE_BYTES) + frag_addr_B(x);
    }
  // within a k-step fragments are read in the order a0,b0,b1,a1,b2,b3,a2,a3, and the MFMA pairs q = 0..7 consume
  // them in that order
  auto mma2 = [&](int q, bf16x8_t(&fa)[MI], bf16x8_t(&fb)[NJ]) {
    constexpr int ii[16] = {0, 0, 1, 1, 0, 1, 0, 1, 2, 2, 2, 2, 3, 3, 3, 3};
    constexpr int jj[16] = {0, 1, 0, 1, 2, 2, 3, 3, 0, 1, 2, 3, 0, 1, 2, 3};
    mma(ii[2 * q], jj[2 * q], fa, fb);
    mma(ii[2 * q + 1], jj[2 * q + 1], fa, fb);
  };
  auto rfrag_ring = [&](int sa, int sb, int ks, int q, bf16x8_t(&fa)[MI], bf16x8_t(&fb)[NJ]) {
    constexpr int isA[8] = {1, 0, 0, 1, 0, 0, 1, 1};
    constexpr int idx[8] = {0, 0, 1, 1, 2, 3, 2, 3};
    if (isA[q]) fa[idx[q]] = frag_A(smem + (sa & 1) * TILE_BYTES, ra_addr[sa >> 1], ks, idx[q]);
    else fb[idx[q]] = frag_B(smem + (sb & 1) * TILE_BYTES, rb_addr[sb >> 1], ks, idx[q]);
  };
  // prologue: A0, B0, A1, B1 into slots 0..3
#pragma unroll
  for (int h = 0; h < 4; ++h) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (h & 1) issue_B(q, smem + h * TILE_BYTES); else issue_A(q, smem + h * TILE_BYTES);
    }
    if (h & 1) next_B(); else next_A();
  }
  // A0 and B0 have landed; A1 and B1 stay in flight across the barrier.  (A plain __syncthreads() here
  // makes the compiler wait for every direct-to-LDS load it knows of, i.e. for all four tiles: stamps
  // inside the kernel, 8-9 K clocks to the first MFMA against 5-6 K.)
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(16) : "memory");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int q = 0; q < 8; ++q) rfrag_ring(0, 1, 0, q, xa, xb);
  // K tile t with t mod 5 == tmod (all slot numbers are compile-time constants)
  auto ring_iteration = [&](const int tmod) __attribute__((always_inline)) {
    const int sa = (2 * tmod) % 5, sb = (2 * tmod + 1) % 5;        // this tile
    const int na = (2 * tmod + 2) % 5, nb = (2 * tmod + 3) % 5;    // the next tile
    const int ia = (2 * tmod + 4) % 5;                             // receives A(t+2); B(t+2) goes to sa
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      rfrag_ring(sa, sb, 1, q, ya, yb);
      if (q < 4) issue_A(q, smem + ia * TILE_BYTES);
      mma2(q, xa, xb);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      rfrag_ring(sa, sb, 2, q, xa, xb);
      if (q < 4) issue_A(4 + q, smem + ia * TILE_BYTES);
      mma2(q, ya, yb);
      __builtin_amdgcn_sched_barrier(0);
    }
    next_A();
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      rfrag_ring(sa, sb, 3, q, ya, yb);
      mma2(q, xa, xb);
      __builtin_amdgcn_sched_barrier(0);
    }
    // A(t+1) and B(t+1) have landed (only the loads of A(t+2) may be pending) and nobody reads
    // this tile's slots any more
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(8) : "memory");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      rfrag_ring(na, nb, 0, q, xa, xb);
      issue_B(q, smem + sa * TILE_BYTES);
      mma2(q, ya, yb);
      __builtin_amdgcn_sched_barrier(0);
    }
    next_B();
  };
  int kt = 0;
  for (; kt + 5 <= nk; kt += 5) {
    if (TOUCH && kt <= touch_at && touch_at < kt + 5) touch_epilogue_inputs();
    ring_iteration(0);
    ring_iteration(1);
    ring_iteration(2);
    ring_iteration(3);
    ring_iteration(4);
  }
  if (TOUCH && kt <= touch_at) touch_epilogue_inputs();
  if (kt < nk) ring_iteration(0);
  if (kt + 1 < nk) ring_iteration(1);
  if (kt + 2 < nk) ring_iteration(2);
  if (kt + 3 < nk) ring_iteration(3);
  } else {
  // ---- main loop: STAGES whole K tiles in LDS ---------------------------------------------------
  // K tile t sits in stage t mod STAGES.  One barrier per K tile, before its last k-step: in front of it the load
  // wavefronts have seen tile t + 1 land (the tiles after it stay in flight) and the others have read the last of
  // tile t, so behind it tile t + STAGES is requested into tile t's stage.
  constexpr int S = C::STAGES, STAGE_BYTES = C::A_BYTES + C::B_BYTES, LOADS = LOADS_A + LOADS_B;
  if (load_wave) {
    auto request = [&](const int st) __attribute__((always_inline)) {
#pragma unroll
      for (int q = 0; q < LOADS_A; ++q) issue_A(q, smem + st * STAGE_BYTES);
      next_A();
#pragma unroll
      for (int q = 0; q < LOADS_B; ++q) issue_B(q, smem + st * STAGE_BYTES + C::A_BYTES);
      next_B();
    };
#pragma unroll
    for (int st = 0; st < S; ++st) request(st);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S - 1) * LOADS) : "memory");
    __builtin_amdgcn_s_barrier();
    auto load_iteration = [&](const int st) __attribute__((always_inline)) {
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S - 2) * LOADS) : "memory");
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      request(st);
      __builtin_amdgcn_sched_barrier(0);
    };
    int kt = 0;
    for (; kt + S <= nk; kt += S) {
#pragma unroll
      for (int st = 0; st < S; ++st) load_iteration(st);
    }
#pragma unroll
    for (int st = 0; st < S - 1; ++st)
      if (kt + st < nk) load_iteration(st);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // nothing lands in LDS once the epilogue stages through it
    __syncthreads();
    return;
  }
  constexpr int NMMA = MI * NJ, NFRAG = MI + NJ;
  uint32_t sa_addr[S][4], sb_addr[S][4];
#pragma unroll
  for (int st = 0; st < S; ++st)
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      sa_addr[st][x] = (uint32_t)(st * STAGE_BYTES) + frag_addr_A(x);
      sb_addr[st][x] = (uint32_t)(st * STAGE_BYTES + C::A_BYTES) + frag_addr_B(x);
    }
  auto rfrag = [&](int st, int ks, int q, bf16x8_t(&fa)[MI], bf16x8_t(&fb)[NJ]) {   // order a0, b0, b1, .., a1, a2, ..
    if (q == 0) fa[0] = frag_A(smem, sa_addr[st], ks, 0);
    else if (q <= NJ) fb[q - 1] = frag_B(smem, sb_addr[st], ks, q - 1);
    else fa[q - NJ] = frag_A(smem, sa_addr[st], ks, q - NJ);
  };
  // one k-step: its MFMAs, with the fragment reads of the next k-step between them
  auto kstep = [&](int st, int ks_next, bf16x8_t(&fa)[MI], bf16x8_t(&fb)[NJ], bf16x8_t(&na)[MI],
                   bf16x8_t(&nb)[NJ]) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < NMMA; ++u) {
#pragma unroll
      for (int q = u * NFRAG / NMMA; q < (u + 1) * NFRAG / NMMA; ++q) rfrag(st, ks_next, q, na, nb);
      mma(u / NJ, u % NJ, fa, fb);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int q = 0; q < NFRAG; ++q) rfrag(0, 0, q, xa, xb);
  auto stage_iteration = [&](const int st) __attribute__((always_inline)) {
    kstep(st, 1, xa, xb, ya, yb);
    kstep(st, 2, ya, yb, xa, xb);
    kstep(st, 3, xa, xb, ya, yb);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    kstep((st + 1) % S, 0, ya, yb, xa, xb);
  };
  int kt = 0;
  for (; kt + S <= nk; kt += S) {
    if (TOUCH && kt <= touch_at && touch_at < kt + S) touch_epilogue_inputs();
#pragma unroll
    for (int st = 0; st < S; ++st) stage_iteration(st);
  }
  if (TOUCH && kt <= touch_at) touch_epilogue_inputs();
#pragma unroll
  for (int st = 0; st < S - 1; ++st)
    if (kt + st < nk) stage_iteration(st);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (TOUCH)   // end of the touched registers' reservation
#pragma unroll
    for (int x = 0; x < MI; ++x) asm volatile("" ::"v"(touched[x]));
  __syncthreads();

  // ---- epilogue: per wavefront, 32 rows at a time through LDS ----------------------------
  constexpr int SROW = WSN * 4 + 16;           // staged row: fp32 values + 16 bytes of padding
  constexpr int OUTW = DUAL ? WSN / 2 : WSN;  // output columns of a wavefront
  constexpr int LPR = OUTW / 8;               // lanes per row, 8 columns each
  constexpr int RPP = 64 / LPR;               // rows per pass of the wavefront
  constexpr int PASSES = 32 / RPP;
  char* stg = smem + wave * (32 * SROW);
  const int srow = lane / LPR;                // row within a pass
  const int scol = (lane & (LPR - 1)) * 8;    // first of this lane's 8 consecutive columns
  const int n = n0 + wn * OUTW + scol;
  const bool n_ok = n < p.N;
  const int n_ld = n_ok ? n : 0;              // in-bounds column for the prefetching loads
  constexpr bool GATE_LIKE = (EPI == EPI_GATE || EPI == EPI_GATE_UP || EPI == EPI_GATE_UPE || DUAL);
  constexpr bool DH_LIKE = (EPI == EPI_DH || EPI == EPI_DH_UP || EPI == EPI_DH_UPE);
  constexpr bool USE_E = (EPI == EPI_GATE || EPI == EPI_DH || EPI == EPI_GATE_UPE || EPI == EPI_DH_UPE || EPI == EPI_GATE_DUALE);
  constexpr bool USE_UP = (EPI == EPI_GATE_UP || EPI == EPI_GATE_UPE || EPI == EPI_DH_UP || EPI == EPI_DH_UPE);
  constexpr bool FUSED = GATE_LIKE || DH_LIKE;

  // Everything the element-wise part needs from memory is requested one 32-row block ahead
  // (PASSES rows per lane and block), so the gathered table rows arrive while the previous block
  // is being staged and stored.
  // ev: gathered table row, uv: up-projection row (dense and additive variants), gv: saved G row
  uint4 ev[2][PASSES], gv[2][PASSES], uv[2][PASSES];
  // The backward pass reads the saved G and Up once, so there they are read past the caches and leave the room to dU, dG and the operand
  // panels (whole training steps, us, kept / past: 3000 tokens of a dense 1536 x 5120 layer 450 / 435; 4096 of an additive 1024 x 4096
  // layer, 1999 of 2048 x 8192, 600 of 1536 x 5120 and 5000 of 640 x 2048 the same within what runs differ by, 1 to 2 %.  G stored past them as well: 1999
  // tokens 457 against 459, but 640 x 2048 174 against 172; dU too: 600 of 1536 x 5120 132.5 against 130.3).
  auto load_once = [](const bf16_t* at) __attribute__((always_inline)) {
    if (!DH_LIKE) return *reinterpret_cast<const uint4*>(at);
    return __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(at)));
  };
  auto prefetch = [&](int i, int buf) __attribute__((always_inline)) {
    if (!FUSED) return;
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) {
      const int m = m0 + wm * WSM + i * 32 + pass * RPP + srow;
      const int mc = m < p.M ? m : p.M - 1;
      if (USE_E) {
        const int r = i * 32 + pass * RPP + srow;   // row within the wavefront's quadrant: held by lane r & 63
        const int id = __builtin_amdgcn_ds_bpermute((r & 63) * 4, row_id[i >> 1]);
        ev[buf][pass] = *reinterpret_cast<const uint4*>(p.E + (size_t)id * p.N + n_ld);
      }
      if (USE_UP) uv[buf][pass] = load_once(p.inUp + (size_t)mc * p.N + n_ld);
      if (DH_LIKE) gv[buf][pass] = load_once(p.inG + (size_t)mc * p.N + n_ld);
    }
  };
  // Outputs leave through buffer stores: a lane outside the matrix (ragged last tile) is given an
  // offset beyond the buffer and the hardware drops its store, so the element-wise part below is
  // straight-line code that the compiler schedules as a whole (the staged values of all
  // passes are read from LDS up front and the arithmetic of one pass covers the latency of the
  // next; with a branch around every store each pass waited for its own LDS reads: stamps inside
  // the kernel, 5.7 K clocks per 32-row block against 3.6 K of arithmetic).
  auto out_rsrc = [&](void* ptr, int esize) {
    return __builtin_amdgcn_make_buffer_rsrc(ptr, 0, ptr ? (int)((int64_t)p.M * p.N * esize) : 0, 0x00020000);
  };
  rsrc_t r0, r1;   // EPI_BF16 / EPI_F32: C;  gate-like: G (may be absent), H;  dH-like: dU, dG
  if (EPI == EPI_BF16) r0 = r1 = out_rsrc(p.C, 2);
  else if (EPI == EPI_BF16_RES) { r0 = out_rsrc(p.C, 2); r1 = out_rsrc(const_cast<bf16_t*>(p.residual), 2); }
  else if (EPI == EPI_F32) r0 = r1 = out_rsrc(p.C, 4);
  else if (GATE_LIKE) { r0 = out_rsrc(p.outG, 2); r1 = out_rsrc(p.outH, 2); }
  else { r0 = out_rsrc(p.outdU, 2); r1 = out_rsrc(p.outdG, 2); }
  auto store16 = [&](rsrc_t r, uint32_t off, uint4 v) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v), r, off, 0, 0);
  };
  prefetch(0, 0);
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    if (i + 1 < MI) prefetch(i + 1, (i + 1) & 1);
    // accumulators -> LDS: lane holds row frow, columns j*32 + g*8 + fk*4 .. +3
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const f32x16_t v = acc[i][j];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        f32x4_t w = {v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
        *reinterpret_cast<f32x4_t*>(stg + frow * SROW + (j * 32 + g * 8 + fk * 4) * 4) = w;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    f32x4_t cv[PASSES][2];
    f32x4_t cu[DUAL ? PASSES : 1][2];
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) {
      const int r = pass * RPP + srow;
      cv[pass][0] = *reinterpret_cast<const f32x4_t*>(stg + r * SROW + scol * 4);
      cv[pass][1] = *reinterpret_cast<const f32x4_t*>(stg + r * SROW + scol * 4 + 16);
      if constexpr (DUAL) {
        cu[pass][0] = *reinterpret_cast<const f32x4_t*>(stg + r * SROW + (OUTW + scol) * 4);
        cu[pass][1] = *reinterpret_cast<const f32x4_t*>(stg + r * SROW + (OUTW + scol) * 4 + 16);
      }
    }
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) {
      const int r = pass * RPP + srow;
      const int m = m0 + wm * WSM + i * 32 + r;
      const f32x4_t c0 = cv[pass][0], c1 = cv[pass][1];
      const float c[8] = {c0[0], c0[1], c0[2], c0[3], c1[0], c1[1], c1[2], c1[3]};
      const bool ok = n_ok && m < p.M;
      const uint32_t o = ok ? (uint32_t)m * (uint32_t)p.N + (uint32_t)n : 0u;   // element index, < 2^30
      const uint32_t o2 = ok ? o * 2u : OOB, o4 = ok ? o * 4u : OOB;
      if (EPI == EPI_BF16) {
        store16(r0, o2, pack8(c));
      } else if (EPI == EPI_BF16_RES) {
        float rz[8], sum[8];
        unpack8(__builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r1, o2, 0, 0)), rz);
#pragma unroll
        for (int q = 0; q < 8; ++q) sum[q] = c[q] + rz[q];
        store16(r0, o2, pack8(sum));
      } else if (EPI == EPI_F32) {
        // the previous value is fetched only when it is to be added to: otherwise the load is out of range and reads zero
        const uint32_t ol = p.accumulate ? o4 : OOB;
        const u32x4_t q0 = __builtin_amdgcn_raw_buffer_load_b128(r0, ol, 0, 0);
        const u32x4_t q1 = __builtin_amdgcn_raw_buffer_load_b128(r0, ol, 16, 0);
        const f32x4_t a0 = __builtin_bit_cast(f32x4_t, q0), a1 = __builtin_bit_cast(f32x4_t, q1);
        const f32x4_t v0 = {c[0] + a0[0], c[1] + a0[1], c[2] + a0[2], c[3] + a0[3]};
        const f32x4_t v1 = {c[4] + a1[0], c[5] + a1[1], c[6] + a1[2], c[7] + a1[3]};
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v0), r0, o4, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v1), r0, o4, 16, 0);
      } else {
        // e: what SiLU(G) is multiplied by: the gathered row, the up projection, or their sum
        float e[8];
        if (USE_E) unpack8(ev[i & 1][pass], e);
        if (USE_UP) {
          float u[8];
          unpack8(uv[i & 1][pass], u);
#pragma unroll
          for (int q = 0; q < 8; ++q) e[q] = USE_E ? e[q] + u[q] : u[q];
        }
        if constexpr (DUAL) {   // Up as it is stored, in front of G and H, which may lie over it
          const f32x4_t u0 = cu[pass][0], u1 = cu[pass][1];
          float u[8] = {u0[0], u0[1], u0[2], u0[3], u1[0], u1[1], u1[2], u1[3]};
          const uint4 up = pack8(u);
          store16(out_rsrc(p.outUp, 2), o2, up);
          unpack8(up, u);
#pragma unroll
          for (int q = 0; q < 8; ++q) e[q] = USE_E ? e[q] + u[q] : u[q];
        }
        if (GATE_LIKE) {
          float h[8];
#pragma unroll
          for (int q = 0; q < 8; ++q) h[q] = c[q] * sigmoidf_fast(c[q]) * e[q];
          store16(r0, o2, pack8(c));      // dropped by the hardware when G is not wanted (zero-sized buffer)
          store16(r1, o2, pack8(h));
        } else {  // dH product
          float gz[8], du[8], dg[8];
          unpack8(gv[i & 1][pass], gz);
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            // dU = C SiLU(G) = C g s;  dG = C e SiLU'(G) = C e s (1 + g (1 - s)) = e (dU (1 - s) + C s)
            const float sg = sigmoidf_fast(gz[q]);
            const float cs = c[q] * sg;
            du[q] = cs * gz[q];
            dg[q] = e[q] * fmaf(du[q], 1.0f - sg, cs);
          }
          store16(r0, o2, pack8(du));
          store16(r1, o2, pack8(dg));
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// C[i] = (accumulate ? C[i] : 0) + (sum over the K slices, in slice order, of ws[z][i]); 4 elements per thread
struct SumOut { float* C[3]; int64_t end[3]; };   // the products' outputs, and where each ends in a slice
__global__ __launch_bounds__(256) void splitk_sum_f32_kernel(const float* __restrict__ ws, int ksplit, int64_t total,
                                                             SumOut out, int accumulate) {
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= total) return;
  float* const C = i < out.end[0] ? out.C[0] : i < out.end[1] ? out.C[1] - out.end[0] : out.C[2] - out.end[1];
  f32x4_t s = *reinterpret_cast<const f32x4_t*>(ws + i);
  for (int z = 1; z < ksplit; ++z) s += *reinterpret_cast<const f32x4_t*>(ws + (size_t)z * total + i);
  if (accumulate) s += *reinterpret_cast<const f32x4_t*>(C + i);
  *reinterpret_cast<f32x4_t*>(C + i) = s;
}

// ---- choice of the tiling and of the K split ----------------------------------------------------
// A launch is priced as rounds of 256 workgroups: a round takes (K tiles per workgroup) x (time per K tile) plus a
// fixed part (prologue, epilogue).  The time per K tile grows with the share of the chip that is busy (operand
// loads, clock), from `idle` with a few workgroups to `full` with 256, in the first round and in what is left for the
// last: the chip is power-limited, and a last round with few workgroups runs at a higher clock.  The constants (us) are
// chosen for what the choice loses against the best of the tilings and splits, over every product of forward and backward
// of 237 layers (d_model 512 to 2048, d_ff 2.5 to 4 times that, 130 to 65536 tokens, with and without up projection): 0.3 %
// in the mean, more than 5 % at 55 of 3204.  (With the last round at the full time, and constants fitted to two widths:
// 0.7 %, 172 of 3204, the dearest of them 256x128 tiles where 256x256 ones end in half a round: gate product 1280 x 3328,
// 16384 tokens, 180 us against 166; dx of the layer with up projection, 1536 x 5120, 24000 tokens, 732 against 646.)
// Examples, us (Tile256 / Tile256x128 / Tile128): down product 2048 x 8192, 1999 tokens 146 / 92 / 70, 4096 tokens
// 165 / 114 / 129, 16384 tokens 408 / 460 / 538; gate product 700 tokens 51 / 34 / 39, 1999 tokens 69 / 73 / 85.
struct TilingCost { int tm, tn; double idle, full, fixed_plain, fixed_fused, fixed_f32; };
constexpr TilingCost kTilings[4] = {{256, 256, 0.86, 1.39, 9, 21, 17.5}, {256, 128, 0.45, 0.86, 6, 11, 11}, {128, 128, 0.34, 0.56, 4, 6.5, 5.5}, {192, 128, 0.33, 0.69, 4.5, 8.5, 8}};

struct Plan { int tiling, ksplit; double us; };

// fused: the epilogue carries the layer's element-wise work and cannot be split.  ops: operand pairs of the K range
// (each pair is cut into the same number of slices).  Slices of which the last ones would be left without a K tile (33 K
// tiles in 8 slices of 5) become as many as have one.  n: products in the launch, of M x N outputs or N x M.
Plan choose_plan(int M, int N, int K, int ops, bool fused, bool f32, size_t ws_bytes, int n = 1, const bool* turned = nullptr) {
  Plan best = {0, 1, 1e30};
  const int nk = ops * ((K + BK - 1) / BK);
  for (int t = 0; t < 4; ++t) {
    if (t == 3 && (f32 || ops > 1)) break;
    const TilingCost& c = kTilings[t];
    double tiles = 0;
    for (int q = 0; q < n; ++q) {
      const int m = turned && turned[q] ? N : M, w = turned && turned[q] ? M : N;
      tiles += (double)((m + c.tm - 1) / c.tm) * ((w + c.tn - 1) / c.tn);
    }
    for (int ks = 1; ks <= 8; ks *= 2) {
      if (ks > 1 && (fused || (double)M * N * n * 4 * ks > (double)ws_bytes || nk / ks < 4 || tiles * ks > 512)) break;
      int kt = nk, slices = 1;
      if (ks > 1) {
        kt = (nk + ks - 1) / ks;
        slices = ops * ((nk / ops + kt - 1) / kt);
      }
      // 192x128 tiles where they make one round and fill it, K is more than 8 K tiles (512: 3 to 5 % slower than 256x128) and
      // slices are long enough to be worth their sum; at least 4 % below the others, for what the model is off.
      if (t == 3 && (tiles * slices > 256 || tiles * slices <= 224 || nk <= 8 || (ks > 1 && kt < 32))) continue;
      const double wgs = tiles * slices, fixed = fused ? c.fixed_fused : f32 || ks > 1 ? c.fixed_f32 : c.fixed_plain;
      const int rounds = (int)(wgs / 256);
      const double rest = wgs - rounds * 256.0;
      double us = rounds * (kt * c.full + fixed);
      if (rest > 0) us += kt * (c.idle + (c.full - c.idle) * rest / 256) + fixed;
      if (ks > 1) us += 3 + (slices + 1.0) * M * N * n * 4 / 4.2e6;   // the kernel that sums the slices: launch, and 4.2 TB/s
      if (us * (t == 3 ? 1.04 : 1.0) < best.us) best = {t, slices, us};
    }
  }
  return best;
}

int grid_of(const GemmArgs& a, int tm, int tn) {
  int tiles = ((a.M + tm - 1) / tm) * ((a.N + tn - 1) / tn);
  for (int e = 0; e < a.n_more; ++e) tiles += ((a.more[e].M + tm - 1) / tm) * ((a.more[e].N + tn - 1) / tn);
  return tiles * a.ksplit;
}

template <class C, int LA, int LB, int EPI>
hipError_t launch_tiles(stem_ctx* ctx, int kid, const GemmArgs& a, hipStream_t s) {
  ProfScope ps(ctx, kid, s);
  hipLaunchKernelGGL((gemm_bf16_kernel<C, LA, LB, EPI>), dim3(grid_of(a, C::TM, EPI == EPI_GATE_DUAL || EPI == EPI_GATE_DUALE ? C::TN / 2 : C::TN)), dim3((C::WAVES + C::LW) * 64), 0, s, a);
  return hipGetLastError();
}

template <int LA, int LB, int EPI>
hipError_t launch_tiling(int tiling, stem_ctx* ctx, int kid, const GemmArgs& a, hipStream_t s) {
  if constexpr (LA == OP_KC)   // a rows-contiguous operand's K rows do not divide 192 rows into loads
    if (tiling == 3) return launch_tiles<Tile192x128, LA, LB, EPI>(ctx, kid, a, s);
  if (tiling == 2) return launch_tiles<Tile128, LA, LB, EPI>(ctx, kid, a, s);
  if (tiling == 1) return launch_tiles<Tile256x128, LA, LB, EPI>(ctx, kid, a, s);
  return launch_tiles<Tile256, LA, LB, EPI>(ctx, kid, a, s);
}

hipError_t sum_slices_f32(stem_ctx* ctx, const GemmArgs& a, hipStream_t s) {
  SumOut out;
  int64_t end = 0;
  for (int e = 0; e < 3; ++e) {
    if (e <= a.n_more) end += e == 0 ? (int64_t)a.M * a.N : (int64_t)a.more[e - 1].M * a.more[e - 1].N;
    out.C[e] = static_cast<float*>(e == 0 || e > a.n_more ? a.C : a.more[e - 1].C);
    out.end[e] = end;
  }
  ProfScope ps(ctx, K_SPLITK_REDUCE, s);
  hipLaunchKernelGGL(splitk_sum_f32_kernel, dim3((unsigned)((a.elems / 4 + 255) / 256)), dim3(256), 0, s, a.ws, a.ksplit,
                     a.elems, out, a.accumulate);
  return hipGetLastError();
}

template <int LA, int LB, int EPI>
hipError_t launch(stem_ctx* ctx, int kid, GemmArgs a, hipStream_t s) {
  constexpr bool PLAIN = (EPI == EPI_BF16 || EPI == EPI_BF16_RES), F32 = (EPI == EPI_F32);
  const size_t ws_bytes = a.ws && (int64_t)a.M * a.N % 4 == 0 && (!a.A2 || a.K2 == a.K) ? a.ws_bytes : 0;
  constexpr int WIDTH = EPI == EPI_GATE_DUAL || EPI == EPI_GATE_DUALE ? 2 : 1;
  const Plan plan = choose_plan(a.M, a.N * WIDTH, a.K, a.A2 ? 2 : 1, !PLAIN && !F32, F32, ws_bytes);
  a.ksplit = plan.ksplit;
  a.elems = (int64_t)a.M * a.N;
  if constexpr (PLAIN || F32) {
    if (plan.ksplit > 1) {   // fp32 partial products, one per K slice, and a kernel that sums them in slice order
      hipError_t e = launch_tiling<LA, LB, EPI_F32>(plan.tiling, ctx, kid, a, s);
      if (e != hipSuccess) return e;
      if (PLAIN) return stem_splitk_reduce(ctx, a.ws, plan.ksplit, a.elems, EPI == EPI_BF16_RES ? a.residual : nullptr, a.C, s);
      return sum_slices_f32(ctx, a, s);
    }
  }
  return launch_tiling<LA, LB, EPI>(plan.tiling, ctx, kid, a, s);
}

}  // namespace

void stem_route_tiles(int M, int N, int K, int ops, int epi, int64_t ws_bytes, int32_t* route) {
  const bool plain = epi == EPI_BF16 || epi == EPI_BF16_RES;
  const Plan p = choose_plan(M, N, K, ops, !plain && epi != EPI_F32, epi == EPI_F32, (size_t)ws_bytes);
  route[0] = ROUTE_TILES; route[1] = kTilings[p.tiling].tm; route[2] = kTilings[p.tiling].tn; route[3] = p.ksplit;
}

hipError_t stem_gemm_bf16(stem_ctx* ctx, int kid, int la, int lb, int epi, const GemmArgs& a, hipStream_t s) {
  if (a.M <= 0 || a.N <= 0 || a.K <= 0) return hipSuccess;
  // buffer offsets are 32-bit: every operand must stay below 2 GiB
  const int64_t lim = 0x7fffffff;
  const int64_t abytes = (la == OP_KC ? (int64_t)a.M : (int64_t)a.K) * a.lda * 2;
  const int64_t bbytes = (lb == OP_KC ? (int64_t)a.N : (int64_t)std::max(a.K, a.K2)) * a.ldb * 2;
  if (abytes > lim || bbytes > lim) return hipErrorInvalidValue;
  if (a.A2 && la != OP_KC) return hipErrorInvalidValue;   // a second operand pair needs a K-contiguous A
  // so are the outputs' (buffer stores)
  if ((int64_t)a.M * a.N * (epi == EPI_F32 ? 4 : 2) > lim) return hipErrorInvalidValue;
  if (la == OP_KC && lb == OP_KC) {
    if (epi == EPI_BF16) return launch<OP_KC, OP_KC, EPI_BF16>(ctx, kid, a, s);
    if (epi == EPI_BF16_RES) return launch<OP_KC, OP_KC, EPI_BF16_RES>(ctx, kid, a, s);
    if (epi == EPI_GATE) return launch<OP_KC, OP_KC, EPI_GATE>(ctx, kid, a, s);
    if (epi == EPI_GATE_UP) return launch<OP_KC, OP_KC, EPI_GATE_UP>(ctx, kid, a, s);
    if (epi == EPI_GATE_UPE) return launch<OP_KC, OP_KC, EPI_GATE_UPE>(ctx, kid, a, s);
    if (epi == EPI_GATE_DUAL) return launch<OP_KC, OP_KC, EPI_GATE_DUAL>(ctx, kid, a, s);
    if (epi == EPI_GATE_DUALE) return launch<OP_KC, OP_KC, EPI_GATE_DUALE>(ctx, kid, a, s);
  } else if (la == OP_KC && lb == OP_MC) {  // activation gradients: the weight as stored, rows-contiguous
    if (epi == EPI_BF16) return launch<OP_KC, OP_MC, EPI_BF16>(ctx, kid, a, s);
    if (epi == EPI_DH) return launch<OP_KC, OP_MC, EPI_DH>(ctx, kid, a, s);
    if (epi == EPI_DH_UP) return launch<OP_KC, OP_MC, EPI_DH_UP>(ctx, kid, a, s);
    if (epi == EPI_DH_UPE) return launch<OP_KC, OP_MC, EPI_DH_UPE>(ctx, kid, a, s);
  } else if (la == OP_MC && lb == OP_MC) {  // weight gradients: both operands [K, rows], rows contiguous
    if (epi == EPI_F32) return launch<OP_MC, OP_MC, EPI_F32>(ctx, kid, a, s);
  }
  return hipErrorInvalidValue;
}

// Weight gradients of one K whose tiles leave part of the chip idle, or need K slices to fill it, share a launch: fewer
// slices (whose partial products cost as much to sum as to write), one prologue and epilogue per round instead of one per
// product, and one last round.  Taken where the cost model prices the one launch 4 % below the several, and 3 us for each launch
// saved.  Where tiles, slices and rounds stay the same, up to 250 us: beyond, the saved launches are worth less than what the
// products lose that the XCDs then read the operands of two or three of them at a time, and dx and dW_gate that dG was not read
// just before.  Backward, us, apart / together: 1920 x 6400, 1013 tokens 130 / 126; 1984 x 7296, 5702 tokens 604 / 599; 1344 x
// 5312 with an up projection, 6773 tokens 601 / 617, 1472 x 3840, 7961 tokens 542 / 568; 1792 x 7104, 21592 tokens 1915 / 1952;
// 2048 x 8192, 16384 tokens 1704 / 1709.  With fewer rounds or slices: 1024 x 4096, 16384 tokens 541 / 508; with an up
// projection, 4096 tokens 225 / 211.  Over 260 layers (d_model 512 to 2048, 128 to 65536 tokens) the rule takes 0.895 of the
// time that launches of their own take, with an up projection 0.862, and loses 1.1 % at worst.
//
// Fewer slices are sums of twice the length, or four times: a gradient's distance from the exact sum of the same bf16 operands
// goes from 4.1e-7 to 5.8e-7 of it (1024 x 4096, 16384 tokens), from 3.7e-7 to 7.6e-7 (640 x 2496 with an up projection, 14279
// tokens; 1472 x 5568, never cut, has 8.3e-7 at 16768).  Its distance from the layer's in 64 bits, 1.6587e-3 from the rounding of
// H or dG to bf16, is the same to six digits.
static bool plan_together(const GemmArgs* a, int n, size_t ws_bytes, GroupPlan* plan) {
  bool turned[3] = {}, alike = n == 2 || n == 3;
  double apart = 0;
  Plan one[3] = {};
  for (int e = 0; e < n && alike; ++e) {
    turned[e] = a[e].M != a[0].M;
    alike = a[e].K == a[0].K && a[e].accumulate == a[0].accumulate &&
            (turned[e] ? a[e].M == a[0].N && a[e].N == a[0].M : a[e].N == a[0].N);
    one[e] = choose_plan(a[e].M, a[e].N, a[e].K, 1, false, true, ws_bytes);
    apart += one[e].us;
  }
  if (!alike) return false;
  const Plan p = choose_plan(a[0].M, a[0].N, a[0].K, 1, false, true, ws_bytes, n, turned);
  *plan = {p.tiling, p.ksplit};
  bool whole = p.us <= apart * 1.0001 && p.us <= 250;   // the same rounds, one after another
  for (int e = 0; e < n; ++e) whole = whole && one[e].tiling == p.tiling && one[e].ksplit == p.ksplit;
  return whole || p.us <= 0.96 * apart + 3 * (n - 1);
}

void stem_route_weight_grads(int d, int F, int64_t T, int n, int64_t ws_bytes, int32_t* route) {
  GemmArgs a[3] = {};
  for (int e = 0; e < 3; ++e) { a[e].M = e ? F : d; a[e].N = e ? d : F; a[e].K = (int)T; }
  GroupPlan plan = {};
  route[0] = plan_together(a, n, (size_t)ws_bytes, &plan);
  route[1] = kTilings[plan.tiling].tm; route[2] = kTilings[plan.tiling].tn; route[3] = plan.ksplit;
}

int stem_route_tile(const int32_t* M, const int32_t* N, int n, int tile_rows, int tile_cols, int band, int ksplit, int block, int32_t* at) {
  GemmArgs a = {};
  a.M = M[0]; a.N = N[0]; a.ksplit = ksplit; a.n_more = n - 1;
  for (int e = 1; e < n; ++e) { a.more[e - 1].M = M[e]; a.more[e - 1].N = N[e]; }
  int tiles[2] = {};
  for (int e = 0; e < 2 && e < n; ++e) tiles[e] = ((M[e] + tile_rows - 1) / tile_rows) * ((N[e] + tile_cols - 1) / tile_cols);
  const int grid = grid_of(a, tile_rows, tile_cols);
  const Place q = place_of(block, grid, ksplit, a.n_more, tiles[0], tiles[1]);
  at[0] = q.product; at[1] = q.slice;
  tile_at(band, q.in, (M[q.product] + tile_rows - 1) / tile_rows, (N[q.product] + tile_cols - 1) / tile_cols, at[2], at[3]);
  return grid;
}

bool stem_weight_grads_together(const GemmArgs* a, int n, GroupPlan* plan) {
  const int64_t lim = 0x7fffffff;   // operands and outputs below 2 GiB, as for each product by itself
  for (int e = 0; e < n; ++e)
    if (a[e].M <= 0 || a[e].N <= 0 || a[e].K <= 0 || (int64_t)a[e].K * a[e].lda * 2 > lim || (int64_t)a[e].K * a[e].ldb * 2 > lim ||
        (int64_t)a[e].M * a[e].N * 4 > lim)
      return false;
  return plan_together(a, n, a[0].ws && (int64_t)a[0].M * a[0].N % 4 == 0 ? a[0].ws_bytes : 0, plan);
}

hipError_t stem_weight_grads(stem_ctx* ctx, const GemmArgs* a, int n, const GroupPlan& plan, hipStream_t s) {
  GemmArgs g = a[0];
  g.n_more = n - 1;
  for (int e = 1; e < n; ++e) g.more[e - 1] = {a[e].A, a[e].B, a[e].C, a[e].M, a[e].N, a[e].lda, a[e].ldb};
  g.ksplit = plan.ksplit;
  g.elems = (int64_t)g.M * g.N * n;
  const hipError_t r = launch_tiling<OP_MC, OP_MC, EPI_F32>(plan.tiling, ctx, K_GEMM_DW, g, s);
  return r != hipSuccess || g.ksplit == 1 ? r : sum_slices_f32(ctx, g, s);
}
