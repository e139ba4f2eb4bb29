// bf16 GEMM on the gfx950 matrix cores (v_mfma_f32_16x16x32_bf16), fp32 accumulate.
//
// One workgroup computes a BM x BN tile of C, stepping BK = 64 along K.  Each step's A and
// B tiles are copied global -> registers -> LDS (16-byte buffer loads, double-buffered LDS, the
// loads of tile kt+2 in flight during the MFMAs of tile kt).  Operands whose
// global layout is K-contiguous sit in LDS as [row][BK] with the 16-byte chunk index
// XOR-swizzled by row bits (conflict-free ds_read_b128 of MFMA fragments on the 64-bank LDS).  Operands whose
// global layout has K as the slow dimension (B of the forward product, both operands of
// the weight-gradient product) sit in LDS as [BK][cols + pad] and are read through the
// LDS transpose load (ds_read_b64_tr_b16), which hands every lane four consecutive k of
// its own column: no transposed copy of any tensor is ever made in HBM.
//
// Wave w of the workgroup owns a (BM / WM) x (BN / WN) sub-tile as MI x NI MFMA tiles of
// 16 x 16 (k = 32 per instruction).  Operand fragment of one MFMA: lane l holds the 8 consecutive
// k from 8 * (l / 16) of row (A) or column (B) l % 16.  Accumulator layout: lane l, register r holds
// row (l / 16) * 4 + r, column l % 16.  The 16 x 16 x 32 form is used because the step runs at the
// socket power limit: in a register-only loop on random operands it sustains 2.00 PFLOP/s where
// the 32 x 32 x 16 form sustains 1.81 (both reach 2.48 on zeros).
#include <atomic>
#include <type_traits>

#include "common.h"
#include "epilogue.h"

namespace bf {

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

constexpr int BK = 64;
// measured throughput of a compute unit on the smaller tiles relative to the 256 x 256 tile
constexpr double TILE_RATE_MID = 0.84, TILE_RATE_SMALL = 0.68, TILE_RATE_WIDE = 0.95;
constexpr int TPAD = 32;  // padding (elements) of a transposed LDS row: stride = 64 bytes mod 128

template <int BM_, int BN_, int WM_, int WN_, int KG_ = 1>
struct Tile {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_;
  static constexpr int KG = KG_;  // groups of WM x WN waves that share the contraction of the tile
  static constexpr int NT = WM * WN * 64;
  static constexpr int TM = BM / WM, TN = BN / WN;
  static constexpr int MI = TM / 16, NI = TN / 16;
  static_assert(MI % 2 == 0, "the A fragments of a k-step are fetched in two halves");
};

// XOR key of a K-contiguous LDS row (128 bytes = 8 chunks of 16 bytes).  The LDS has 64 banks of 4
// bytes and serves a 16-byte-per-lane read 16 lanes at a time, but not 16 consecutive lanes: the
// first cycle of a 32-lane half takes lanes 0-3, 12-15, 20-23, 24-27, the second the other four
// quads (the bank-conflict counter reads zero for layouts that are conflict-free under this
// grouping and a steady two-way conflict for one that is only conflict-free for consecutive lanes).
// A fragment read has lane l at row l % 16 and logical chunk c + l / 16, so one cycle sees the row
// pairs {0,1}, {2,3}, {12,13}, {14,15} at chunk c and {4,5}, {6,7}, {8,9}, {10,11} at chunk c ^ 1 (or the
// reverse).  The key sends the first four pairs to 0..3 and the others to 4..7: both sets are closed
// under ^ 1, so the 16 (row parity, chunk) slots of a cycle are distinct.
__device__ __forceinline__ int kswz(int row) {
  return ((row >> 1) & 1) | (((row >> 3) & 1) << 1) | ((((row >> 2) ^ (row >> 3)) & 1) << 2);
}

// XOR key (in 16-byte chunks) of a transposed LDS row: rows k and k + 8 are read together by the two
// 16-lane groups of a 32-lane half of the transpose load and sit a multiple of 256 bytes apart;
// moving one of them by 16 columns (32 bytes) puts the two groups on disjoint banks.
__device__ __forceinline__ int tkey(int krow) { return ((krow >> 3) & 1) << 1; }

// bytes of one LDS stage of an operand tile with R rows (m or n extent)
template <bool KCONTIG, int R>
constexpr int stage_elems() { return KCONTIG ? R * BK : BK * (R + TPAD); }

// ---- global -> registers: the thread's 16-byte chunks of an operand tile.  Chunk i of a thread
// sits a fixed number of tile rows below chunk 0, so one per-thread byte offset (global) and one
// per-thread element offset (LDS) serve all chunks: every load is "wave-uniform base (scalar
// registers, moved per k-tile and per chunk) + 32-bit lane offset", every LDS store "lane offset
// + immediate".
template <bool KCONTIG, int R, int NT, bool EVEN = KCONTIG || NT % (R / 8) == 0>
struct Stager {
  static constexpr int CHUNKS = R * BK / 8 / NT;
  static constexpr int ROWSTEP = KCONTIG ? NT / 8 : NT / (R / 8);  // tile rows between a thread's chunks
  static_assert(ROWSTEP % 16 == 0, "the swizzle keys must repeat from chunk to chunk");
  u32x4 v[CHUNKS];
  uint32_t goff;  // byte offset of chunk 0 from the tile's first element
  int loff;       // element offset of chunk 0 inside the LDS tile
  int kcol;       // first k of the thread's chunks inside the k-tile (K-contiguous operands)

  __device__ __forceinline__ void init(size_t ld, int tid) {
    kcol = (tid & 7) * 8;
    if (KCONTIG) {
      const int row = tid >> 3, kc = tid & 7;  // 8 chunks per row of BK = 64
      goff = (uint32_t)(((size_t)row * ld + kc * 8) * sizeof(bf16_t));
      loff = row * BK + ((kc ^ kswz(row)) << 3);
    } else {
      const int krow = tid / (R / 8), rc = tid % (R / 8);
      goff = (uint32_t)(((size_t)krow * ld + rc * 8) * sizeof(bf16_t));
      loff = krow * (R + TPAD) + ((rc ^ tkey(krow)) << 3);
    }
  }
  // The same for a tile that may reach past the matrix (R_ext rows / columns, K long): the descriptor ends where the
  // matrix ends, and loads past its end return zero.  That covers rows past R_ext of a K-contiguous operand and rows
  // past K of the other kind; chunks past K of a K-contiguous row are sent past the end; columns past R_ext of a
  // K-slow operand pick up values of the next row, which only reach outputs that are not stored.  The whole offset
  // goes through the lane register: a scalar offset would take part in the range check by subtraction.
  // PAST: k0 may lie behind K.
  template <bool PAST = false>
  __device__ __forceinline__ void load_edge(const bf16_t* __restrict__ g, size_t ld, int r0, int k0, int R_ext, int K) {
    const bf16_t* base = KCONTIG ? g + (size_t)r0 * ld + k0 : g + (size_t)k0 * ld + r0;
    // elements to the end
    const size_t left = KCONTIG ? (size_t)(R_ext - r0) * ld - k0 : PAST && k0 >= K ? 0 : (size_t)(K - k0) * ld - r0;
    const size_t cap = (size_t)0x7fffff00 / sizeof(bf16_t);
    __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)((left < cap ? left : cap) * sizeof(bf16_t)), 0x00020000);
    const uint32_t step = (uint32_t)((size_t)ROWSTEP * ld * sizeof(bf16_t));
    const uint32_t off = KCONTIG && kcol >= K - k0 ? 0x7fffff00u : goff;
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) v[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off + i * step, 0, 0);
  }
  // g: operand base (uniform); r0: first row/col of the tile; k0: first k.  Buffer loads: the
  // descriptor carries the tile's base address, the lane offset is a VGPR, the chunk step an SGPR.
  __device__ __forceinline__ void load(const bf16_t* __restrict__ g, size_t ld, int r0, int k0) {
    const bf16_t* base = KCONTIG ? g + (size_t)r0 * ld + k0 : g + (size_t)k0 * ld + r0;
    __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0x7fffffff, 0x00020000);
    const int step = (int)((size_t)ROWSTEP * ld * sizeof(bf16_t));
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) v[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, goff, i * step, 0);
  }
  __device__ __forceinline__ void store(bf16_t* lds) const {
    constexpr int LSTEP = KCONTIG ? ROWSTEP * BK : ROWSTEP * (R + TPAD);
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) *reinterpret_cast<u32x4*>(lds + loff + i * LSTEP) = v[i];
  }
};

// A transposed tile whose rows (R / 8 chunks) the workgroup's threads do not divide into whole passes (192 columns:
// 24 chunks per k-row, 512 threads): the tile's chunks are dealt out in their linear order, chunk tid + i * NT to
// thread tid, and a thread keeps one global and one LDS offset per chunk (they sit in different rows and columns).
template <int R, int NT>
struct Stager<false, R, NT, false> {
  static constexpr int CPR = R / 8;  // chunks per k-row
  static constexpr int CHUNKS = BK * CPR / NT;
  static_assert(BK * CPR % NT == 0, "the tile's chunks must divide among the threads");
  u32x4 v[CHUNKS];
  uint32_t goff[CHUNKS];
  int loff[CHUNKS];

  __device__ __forceinline__ void init(size_t ld, int tid) {
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) {
      const int c = tid + i * NT, krow = c / CPR, rc = c % CPR;
      goff[i] = (uint32_t)(((size_t)krow * ld + rc * 8) * sizeof(bf16_t));
      loff[i] = krow * (R + TPAD) + ((rc ^ tkey(krow)) << 3);
    }
  }
  __device__ __forceinline__ void load(const bf16_t* __restrict__ g, size_t ld, int r0, int k0) {
    const bf16_t* base = g + (size_t)k0 * ld + r0;
    __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0x7fffffff, 0x00020000);
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) v[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, goff[i], 0, 0);
  }
  __device__ __forceinline__ void store(bf16_t* lds) const {
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) *reinterpret_cast<u32x4*>(lds + loff[i]) = v[i];
  }
};

// Lane part of a K-contiguous fragment address, per k-step: the XOR key only has row bits 1-3, which
// come from the lane (fragments start at multiples of 16 rows), so a fragment's address is this
// offset plus a compile-time multiple of 16 rows and every read takes an immediate.
struct KFragLane {
  int o[2];
  __device__ __forceinline__ void init(int lane) {
    const int l15 = lane & 15;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) o[kk] = l15 * BK + (((kk * 4 + (lane >> 4)) ^ kswz(l15)) << 3);
  }
};

// The same for a transposed tile of R columns.  The key (16 columns) depends on the lane's 16-lane
// group only; XORed into the column it moves a fragment that starts at an even multiple of 16
// columns up and one that starts at an odd multiple down, hence one offset per parity.
template <int R>
struct TFragLane {
  int o[2];
  __device__ __forceinline__ void init(int lane) {
    const int t = lane & 15, blk = lane >> 4;
    const int k = 8 * blk + (t >> 2), c4 = 4 * (t & 3);
#pragma unroll
    for (int par = 0; par < 2; ++par) o[par] = k * (R + TPAD) + (((16 * par + c4) ^ (tkey(k) << 3)) - 16 * par);
  }
};

// ---- LDS -> MFMA fragment: 8 consecutive k of row/column (r16 + lane % 16), k-step kk (32 wide)
// r16: first row / column of the fragment relative to lds, a multiple of 16 (lds itself starts at a
// multiple of 32 rows / columns of the tile)
template <bool KCONTIG, int R>
__device__ __forceinline__ bf16x8 load_frag(const bf16_t* lds, int r16, int kk, const KFragLane& kl, const TFragLane<R>& tl) {
  if (KCONTIG) {
    return *reinterpret_cast<const bf16x8*>(lds + r16 * BK + kl.o[kk]);
  } else {
    // one transpose load: the 16 lanes of a group read 4 k-rows x 16 columns, 4 columns each, and
    // every lane receives the 4 k of its own column; two of them give the lane its 8 k
    const bf16_t* p = lds + kk * 32 * (R + TPAD) + r16 + tl.o[(r16 >> 4) & 1];
    typedef s16x4 __attribute__((address_space(3))) * lds_v4;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(p + 4 * (R + TPAD)));  // k + 4: same key
    typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;
    s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, both);
  }
}

// AK: A is K-contiguous in memory (forward, dgrad); BKC: B is K-contiguous (dgrad)
// SEG_POW2: the k-tiles per segment are a power of two (weight gradient only; true for every
// sequence length that is one): the segment of a k-tile is then a shift, not a division, which
// takes 40 scalar instructions out of the loop (0.7-1 % of the product)
// EDGE: the tiles may reach past M, N and K (K-contiguous rows a multiple of 8 long, outputs N % 8 == 0): guarded loads
// (Stager::load_edge) and stores, everything else the same.
template <typename TL, bool AK, bool BKC, int EPI, typename TO, bool SEG_POW2, bool EDGE>
__global__ __launch_bounds__(TL::NT * TL::KG) void gemm_mfma_kernel(int M, int N, int K, const bf16_t* __restrict__ A,
                                                           const bf16_t* __restrict__ B, TO* __restrict__ C,
                                                           const float* __restrict__ bias, const TO* __restrict__ R,
                                                           TO* __restrict__ C2, int accumulate, int tiles_m, int remap,
                                                           int n_seg, size_t seg_a, size_t seg_b, float* __restrict__ colpart,
                                                           int ldk) {
  constexpr int BM = TL::BM, BN = TL::BN, NT = TL::NT, MI = TL::MI, NI = TL::NI, KG = TL::KG;
  constexpr int A_ST = stage_elems<AK, BM>(), B_ST = stage_elems<BKC, BN>();
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  constexpr int STAGE = A_ST + B_ST;  // stage s: A tile at smem + s * STAGE, B tile right after it
  // KG groups of waves, each with its own LDS stages, take every KG-th k-tile of the same output tile
  const int grp = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / NT);
  bf16_t* smem = reinterpret_cast<bf16_t*>(smem_raw) + grp * 2 * STAGE;

  const int tid = KG == 1 ? threadIdx.x : threadIdx.x % NT, lane = tid & 63, w = tid >> 6;
  const int wm = w % TL::WM, wn = w / TL::WM;
  // Workgroups go to the 8 XCDs round-robin and each XCD has its own L2: give XCD x a contiguous
  // range of the tile order, and walk that order in groups of 8 row-tiles so that the ~32
  // workgroups an XCD runs at a time form an 8 x 4 block sharing A row-panels and B column-panels.
  int lin = blockIdx.x;
  if (remap) {
    const int per_xcd = gridDim.x >> 3;
    lin = (lin & 7) * per_xcd + (lin >> 3);
  }
  const int tiles_n = gridDim.x / tiles_m;
  const int in_group = 8 * tiles_n;
  int bm, bn;
  if (remap && tiles_m % 8 == 0) {
    const int gi = lin / in_group, rem = lin % in_group;
    bm = gi * 8 + (rem & 7);
    bn = rem >> 3;
  } else {
    bm = lin % tiles_m;
    bn = lin / tiles_m;
  }
  const int m0 = bm * BM, n0 = bn * BN;
  // ldk: row length of the operands that are stored K-contiguous; equal to K except in a split-K launch, where K is
  // the length of the slice this workgroup contracts over
  const size_t lda = AK ? (size_t)ldk : (size_t)M;   // A stored [M,K] or [K,M]
  const size_t ldb = BKC ? (size_t)ldk : (size_t)N;  // B stored [N,K] or [K,N]
  if constexpr (EPI == E_ACCUM && AK) {
    // Split-K launch of a forward / dgrad product (grid.y slices of K): slice y starts K elements further along the
    // contraction and leaves its fp32 partial result in plane y of C ([slices][M][N]); a second kernel adds the
    // planes in order and applies the epilogue.
    const size_t y = blockIdx.y;
    A += y * (size_t)K;
    B += y * (BKC ? (size_t)K : (size_t)K * N);
    C += y * (size_t)M * N;
  }

  f32x4 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;
  if constexpr (EPI == E_ACCUM) {
    // Accumulating into the main-grad: the accumulators START from the stored values, so the reads
    // of C overlap the first k-tiles and the epilogue is a plain store (read-modify-write at the end
    // would stall every workgroup of the round on HBM latency at once).
    if (accumulate && (KG == 1 || grp == 0)) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const size_t row = m0 + wm * TL::TM + i * 16 + (lane >> 4) * 4 + r;
            const size_t col = n0 + wn * TL::TN + j * 16 + (lane & 15);
            if (!EDGE || (row < (size_t)M && col < (size_t)N)) acc[i][j][r] = C[row * (size_t)N + col];
          }
    }
  }

  Stager<AK, BM, NT> sa;
  Stager<BKC, BN, NT> sb;
  sa.init(lda, tid);
  sb.init(ldb, tid);
  // Residual / pre-activation values the epilogue needs (E_BIAS_RES, E_GELU_BWD): the first half is
  // requested before the last k-tile, when the staging registers are free, so that its HBM latency
  // hides behind that tile's MFMAs instead of stalling every workgroup of the round at once; the
  // second half follows after the main loop, when the fragment registers are free, and arrives
  // while the first passes of the epilogue run.
  constexpr int PR = 64, NQ = PR * BN / 8 / NT;
  constexpr bool HAS_R = EPI == E_BIAS_RES || EPI == E_GELU_BWD;
  bf16x8 rpre[HAS_R ? BM / PR : 1][HAS_R ? NQ : 1];
  auto prefetch_r = [&](auto first_half) {
    if constexpr (HAS_R) {
      constexpr int P0 = decltype(first_half)::value ? 0 : BM / PR / 2, P1 = decltype(first_half)::value ? BM / PR / 2 : BM / PR;
#pragma unroll
      for (int p = P0; p < P1; ++p)
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          const int c = tid + q * NT, lr = c / (BN / 8), lc = (c % (BN / 8)) * 8;
          if (EDGE && (grp != 0 || m0 + p * PR + lr >= M || n0 + lc >= N)) {
#pragma unroll
            for (int e = 0; e < 8; ++e) rpre[p][q][e] = (__bf16)0.f;
            continue;
          }
          rpre[p][q] = *reinterpret_cast<const bf16x8*>(reinterpret_cast<const bf16_t*>(R) + (size_t)(m0 + p * PR + lr) * N + n0 + lc);
        }
    }
  };
  const int nk_seg = EDGE ? (K + BK - 1) / BK : K / BK, nk = (nk_seg * n_seg + KG - 1) / KG;
  // k-tile kt lives in segment kt / nk_seg (one segment unless this is a multi-micro-batch weight gradient)
  // (only the weight-gradient product is launched with segments: the others skip the division)
  constexpr bool SEGS = EPI == E_ACCUM && KG == 1;
  const int seg_shift = __builtin_ctz(nk_seg);
  auto seg_of = [&](int kt) { return SEG_POW2 ? kt >> seg_shift : kt / nk_seg; };
  auto seg_a_of = [&](int kt) { return SEGS ? A + (size_t)seg_of(kt) * seg_a : A; };
  auto seg_b_of = [&](int kt) { return SEGS ? B + (size_t)seg_of(kt) * seg_b : B; };
  auto k0_of = [&](int kt) { return !SEGS ? kt * BK : SEG_POW2 ? (kt & (nk_seg - 1)) * BK : (kt % nk_seg) * BK; };
  auto load_a = [&](int kt) {
    if constexpr (KG > 1) sa.template load_edge<true>(A, lda, m0, (kt * KG + grp) * BK, M, K);
    else if constexpr (EDGE) sa.load_edge(seg_a_of(kt), lda, m0, k0_of(kt), M, K);
    else sa.load(seg_a_of(kt), lda, m0, k0_of(kt));
  };
  auto load_b = [&](int kt) {
    if constexpr (KG > 1) sb.template load_edge<true>(B, ldb, n0, (kt * KG + grp) * BK, N, K);
    else if constexpr (EDGE) sb.load_edge(seg_b_of(kt), ldb, n0, k0_of(kt), N, K);
    else sb.load(seg_b_of(kt), ldb, n0, k0_of(kt));
  };
  {
    // A k-tile is two k-steps of 32; a k-step runs in two phases, one per half of the wave's A
    // fragments (MI / 2 x NI MFMAs each), so that only half of them are live at a time.  Phase p uses
    // A buffer p % 2 and B buffer (p / 2) % 2 and fetches the fragments of phase p + 1 meanwhile.
    // One barrier per k-tile, placed between phases 2 and 3.  By then every wave holds its phase-3
    // fragments of the current stage in registers and has written tile kt+1 into the other stage, so
    // after the barrier phase 3's MFMAs run while the first fragments of the NEXT stage are fetched:
    // no LDS latency is exposed behind the barrier.  Within a phase the scheduler is told to
    // alternate one MFMA with one LDS/global access.
    constexpr int MH = MI / 2;
    static_assert(TL::TM % 32 == 0 && TL::TN % 32 == 0, "a wave's sub-tile starts at a multiple of 32");
    KFragLane kl;
    TFragLane<BM> tla;
    TFragLane<BN> tlb;
    kl.init(lane);
    tla.init(lane);
    tlb.init(lane);
    constexpr int NRA = AK ? MH : 2 * MH, NRB = BKC ? NI : 2 * NI;  // LDS reads of an A half / of B
    constexpr int NMMA = MH * NI;
    bf16x8 af[2][MH], bfr[2][NI];
    auto ldA = [&](int buf, const bf16_t* as, int kk, int half) {
#pragma unroll
      for (int i = 0; i < MH; ++i) af[buf][i] = load_frag<AK, BM>(as + wm * TL::TM * (AK ? BK : 1), (half * MH + i) * 16, kk, kl, tla);
    };
    auto ldB = [&](int buf, const bf16_t* bs, int kk) {
#pragma unroll
      for (int j = 0; j < NI; ++j) bfr[buf][j] = load_frag<BKC, BN>(bs + wn * TL::TN * (BKC ? BK : 1), j * 16, kk, kl, tlb);
    };
    auto mma = [&](int abuf, int bbuf, auto half) {
      constexpr int H = decltype(half)::value;
#pragma unroll
      for (int i = 0; i < MH; ++i)
#pragma unroll
        for (int jj = 0; jj < NI; ++jj) {
          // serpentine: one operand changes from one MFMA to the next, never both (on a register-only
          // loop under the power limit 2 % faster than row-major and 5 % than both changing; inside
          // this kernel the difference is within the noise)
          const int j = (i & 1) ? NI - 1 - jj : jj;
          acc[H * MH + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[abuf][i], bfr[bbuf][j], acc[H * MH + i][j], 0, 0, 0);
        }
    };
    // mask: 0x008 MFMA, 0x100 LDS read, 0x200 LDS write, 0x020 global read
    auto interleave2 = [&](auto nread, auto mask1, auto n1, auto mask2, auto n2) {
      constexpr int NREAD = decltype(nread)::value;
#pragma unroll
      for (int i = 0; i < NMMA; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (i * ((NREAD + NMMA - 1) / NMMA) < NREAD) __builtin_amdgcn_sched_group_barrier(0x100, (NREAD + NMMA - 1) / NMMA, 0);
        if (decltype(n1)::value > 0 && i < decltype(n1)::value)
          __builtin_amdgcn_sched_group_barrier(decltype(mask1)::value, 1, 0);
        if (decltype(n2)::value > 0 && i < decltype(n2)::value)
          __builtin_amdgcn_sched_group_barrier(decltype(mask2)::value, 1, 0);
      }
      __builtin_amdgcn_sched_barrier(0);  // nothing moves across the end of a phase
    };
    typedef std::integral_constant<int, 0x200> MW;
    typedef std::integral_constant<int, 0x020> MG;
    constexpr bool SPLIT = AK;  // staging of A in phase 2 instead of phase 0
    typedef std::integral_constant<int, (SPLIT ? 0 : Stager<AK, BM, NT>::CHUNKS) + Stager<BKC, BN, NT>::CHUNKS> NC0;
    typedef std::integral_constant<int, Stager<AK, BM, NT>::CHUNKS> NC2;
    typedef std::integral_constant<int, 0> N0;
    typedef std::integral_constant<int, NRA> RA;
    typedef std::integral_constant<int, NRA + NRB> RAB;
    typedef std::integral_constant<int, 0> H0;
    typedef std::integral_constant<int, 1> H1;

    load_a(0);
    load_b(0);
    sa.store(smem);
    sb.store(smem + A_ST);
    if (nk > 1) {
      load_a(1);
      load_b(1);
    }
    __syncthreads();
    ldA(0, smem, 0, 0);
    ldB(0, smem + A_ST, 0);
    auto iter = [&](int kt, auto do_store, auto do_load) {
      const int cur = kt & 1;
      const bf16_t* as = smem + cur * STAGE;
      const bf16_t* bs = as + A_ST;
      const bf16_t* an = smem + (cur ^ 1) * STAGE;
      const bf16_t* bn2 = an + A_ST;
      // phase 0: tile kt+1 (in registers since the previous iteration) goes to the other stage.  With
      // a K-contiguous A (forward, dgrad) only its B part: the A part follows in phase 2, the phase with
      // the fewest fragment reads, so that the phases issue about the same number of memory
      // instructions beside their MFMAs (+2-6 % on the forward products; the weight-gradient layout,
      // all transpose loads, is 2 % faster with everything in phase 0).
      ldA(1, as, 0, 1);
      if constexpr (decltype(do_store)::value) {
        if constexpr (!SPLIT) sa.store(smem + (cur ^ 1) * STAGE);
        sb.store(smem + (cur ^ 1) * STAGE + A_ST);
      }
      // the registers are free again as soon as their LDS store has issued: the loads of tile kt+2
      // follow at once, a full k-tile ahead of their use
      if constexpr (decltype(do_load)::value) {
        if constexpr (!SPLIT) load_a(kt + 2);
        load_b(kt + 2);
      }
      mma(0, 0, H0{});
      if constexpr (decltype(do_load)::value) interleave2(RA{}, MW{}, NC0{}, MG{}, NC0{});
      else if constexpr (decltype(do_store)::value) interleave2(RA{}, MW{}, NC0{}, MW{}, N0{});
      else interleave2(RA{}, MW{}, N0{}, MW{}, N0{});
      // phase 1
      ldA(0, as, 1, 0);
      ldB(1, bs, 1);
      mma(1, 0, H1{});
      interleave2(RAB{}, MW{}, N0{}, MW{}, N0{});
      // phase 2
      ldA(1, as, 1, 1);
      if constexpr (SPLIT && decltype(do_store)::value) sa.store(smem + (cur ^ 1) * STAGE);
      if constexpr (SPLIT && decltype(do_load)::value) load_a(kt + 2);
      mma(0, 1, H0{});
      if constexpr (SPLIT && decltype(do_load)::value) interleave2(RA{}, MW{}, NC2{}, MG{}, NC2{});
      else if constexpr (SPLIT && decltype(do_store)::value) interleave2(RA{}, MW{}, NC2{}, MW{}, N0{});
      else interleave2(RA{}, MW{}, N0{}, MW{}, N0{});
      __syncthreads();
      // phase 3, overlapped with the fetch of the next stage's first fragments
      ldA(0, an, 0, 0);
      ldB(0, bn2, 0);
      mma(1, 1, H1{});
      interleave2(RAB{}, MW{}, N0{}, MW{}, N0{});
    };
    int kt = 0;
    for (; kt + 2 < nk; ++kt) iter(kt, std::true_type{}, std::true_type{});
    if (kt + 1 < nk) { iter(kt, std::true_type{}, std::false_type{}); ++kt; }
    prefetch_r(std::true_type{});
    iter(kt, std::false_type{}, std::false_type{});
    prefetch_r(std::false_type{});
    __syncthreads();
  }

  if constexpr (KG > 1) {
    // the other groups hand their sums to the first, lane to lane, added in order; the loop ended on a barrier
    float* hand = reinterpret_cast<float*>(smem_raw);
    static_assert(EDGE && (size_t)(KG - 1) * BM * BN * 4 <= (size_t)KG * 2 * STAGE * sizeof(bf16_t), "the hand-over does not fit");
    if (grp > 0) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) hand[(((grp - 1) * MI + i) * NI + j) * 4 * NT + r * NT + tid] = acc[i][j][r];
    }
    __syncthreads();
    if (grp == 0) {
#pragma unroll
      for (int g = 0; g < KG - 1; ++g)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][r] += hand[((g * MI + i) * NI + j) * 4 * NT + r * NT + tid];
    }
    __syncthreads();
  }
  // (the other groups pass the epilogue's barriers and store nothing)
  if constexpr (EPI == E_ACCUM) {
    // fp32 main-grad: 16 lanes cover 64 contiguous bytes of a row, stored directly
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const size_t row = m0 + wm * TL::TM + i * 16 + (lane >> 4) * 4 + r;
          const size_t col = n0 + wn * TL::TN + j * 16 + (lane & 15);
          if (!EDGE || (grp == 0 && row < (size_t)M && col < (size_t)N)) C[row * (size_t)N + col] = acc[i][j][r];
        }
  } else {
    // bf16 outputs: the fp32 accumulators pass through LDS, 64 tile rows at a time, so that every
    // thread finishes 8 adjacent columns (bias, residual, GeLU in fp32, one rounding) and the
    // global accesses of C, C2 and R are 16 bytes per lane over whole 512-byte row segments.
    constexpr int LDC = BN + 4;
    // (with one group the array itself: behind the other pointer the stores lose their constant addresses)
    float* cs = KG == 1 ? reinterpret_cast<float*>(smem_raw) : reinterpret_cast<float*>(smem);
    static_assert((size_t)PR * LDC * 4 <= 2 * (size_t)STAGE * sizeof(bf16_t), "epilogue staging does not fit");
    // E_GELU_BWD with colpart: the column sums of this tile's (rounded) outputs, i.e. the tile's share of the bias
    // gradient of the linear layer whose pre-activation gradient is being written; a thread keeps the sums of
    // its 8 columns over its rows, the threads of a column group meet in LDS after the last pass
    float csum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int p = 0; p < BM / PR; ++p) {
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int r0 = wm * TL::TM + i * 16;
        if (r0 / PR != p) continue;
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            cs[(r0 % PR + (lane >> 4) * 4 + r) * LDC + wn * TL::TN + j * 16 + (lane & 15)] = acc[i][j][r];
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int c = tid + q * NT, lr = c / (BN / 8), lc = (c % (BN / 8)) * 8;
        const size_t row = m0 + p * PR + lr, col = n0 + lc, idx = row * (size_t)N + col;
        if (EDGE && (grp != 0 || row >= (size_t)M || col >= (size_t)N)) continue;
        float v[8];
        *reinterpret_cast<f32x4*>(v) = *reinterpret_cast<const f32x4*>(cs + lr * LDC + lc);
        *reinterpret_cast<f32x4*>(v + 4) = *reinterpret_cast<const f32x4*>(cs + lr * LDC + lc + 4);
        if constexpr (EPI == E_BIAS || EPI == E_BIAS_RES || EPI == E_BIAS_GELU) {
          const f32x4 b0 = *reinterpret_cast<const f32x4*>(bias + col), b1 = *reinterpret_cast<const f32x4*>(bias + col + 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) { v[e] += b0[e]; v[4 + e] += b1[e]; }
        }
        bf16x8 o;
        if constexpr (EPI == E_BIAS_RES) {
          const bf16x8 rr = rpre[p][q];
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = (__bf16)(v[e] + (float)rr[e]);
        } else if constexpr (EPI == E_GELU_BWD) {
          const bf16x8 rr = rpre[p][q];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            o[e] = (__bf16)(v[e] * gelu_grad_f((float)rr[e]));
            csum[e] += (float)o[e];
          }
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = (__bf16)v[e];
        }
        *reinterpret_cast<bf16x8*>(C + idx) = o;
        if constexpr (EPI == E_BIAS_GELU) {
          bf16x8 g2;
#pragma unroll
          for (int e = 0; e < 8; ++e) g2[e] = (__bf16)gelu_f((float)o[e]);
          *reinterpret_cast<bf16x8*>(C2 + idx) = g2;
        }
      }
      __syncthreads();
    }
    if constexpr (EPI == E_GELU_BWD) {
      if (colpart) {
        // thread tid owns column group tid % (BN / 8) in every pass (NT is a multiple of BN / 8) and the rows
        // tid / (BN / 8) + k * RG: RG partial sums per column, added in ascending order
        constexpr int CGN = BN / 8, RG = NT / CGN;
        static_assert(NT % CGN == 0 && (size_t)RG * BN * 4 <= 2 * (size_t)STAGE * sizeof(bf16_t), "column-sum staging does not fit");
        const int g = tid % CGN, rg = tid / CGN;
#pragma unroll
        for (int e = 0; e < 8; ++e) cs[rg * BN + g * 8 + e] = csum[e];
        __syncthreads();
        for (int c = tid; c < BN; c += NT) {
          if (EDGE && (grp != 0 || n0 + c >= N)) break;
          float t = 0.f;
#pragma unroll 8
          for (int r = 0; r < RG; ++r) t += cs[r * BN + c];
          colpart[(size_t)bm * N + n0 + c] = t;
        }
      }
    }
  }
}

typedef Tile<256, 256, 2, 4> TileBig;    // 8 waves, 128 x 64 per wave (8 x 4 MFMA tiles)
typedef Tile<256, 128, 4, 2> TileMid;    // 8 waves, 64 x 64 per wave
typedef Tile<128, 128, 2, 2> TileSmall;  // 4 waves, 64 x 64 per wave
// 8 waves, 64 x 96 per wave, for outputs of 6144 columns (24 times 256, but 32 times 192): 2048 rows are 256 such
// tiles, one round, where 256 x 256 gives 192.  For the forward and dgrad layouts with the one-output epilogues
// (none, bias, bias + residual); the epilogue that also takes column sums needs the threads to divide into the
// tile's 24 column groups and keeps the other shapes.
typedef Tile<256, 192, 4, 2> TileWide;

// 4 waves, 32 x 32 per wave, for products of few tiles (edge form only)
typedef Tile<64, 64, 2, 2> TileTiny;
// with the contraction shared by two or four groups of waves (key_groups)
typedef Tile<64, 64, 2, 2, 2> TileTiny2;
typedef Tile<64, 64, 2, 2, 4> TileTiny4;
typedef Tile<128, 64, 2, 2, 2> TileTall2;

template <typename TL, bool AK, bool BKC>
constexpr size_t lds_bytes() { return TL::KG * 2 * (size_t)(stage_elems<AK, TL::BM>() + stage_elems<BKC, TL::BN>()) * sizeof(bf16_t); }

template <typename TL, bool AK, bool BKC, int EPI, typename TO, bool EDGE = false, bool SEG_POW2 = false>
bf_status launch(const GemmArgs& a, hipStream_t st) {
  if constexpr (EPI == E_ACCUM && !SEG_POW2 && !EDGE) {
    const int nk_seg = a.K / ((AK && a.k_slices > 1) ? a.k_slices : 1) / BK;
    if ((nk_seg & (nk_seg - 1)) == 0) return launch<TL, AK, BKC, EPI, TO, false, true>(a, st);
  }
  auto kern = gemm_mfma_kernel<TL, AK, BKC, EPI, TO, SEG_POW2, EDGE>;
  constexpr size_t lds = lds_bytes<TL, AK, BKC>();
  // The LDS reservation is a per-device attribute of the kernel: one bit per device and instantiation,
  // set after the call has succeeded (two threads racing here both make the call, which is harmless).
  static std::atomic<uint64_t> attr_set{0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) { set_error("gemm_mfma: no current device"); return BF_EDEVICE; }
  const uint64_t bit = 1ull << (dev & 63);
  if (dev >= 64 || !(attr_set.load(std::memory_order_acquire) & bit)) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) { set_error("gemm_mfma: cannot reserve %zu bytes of LDS: %s", lds, hipGetErrorString(e)); return BF_EDEVICE; }
    if (dev < 64) attr_set.fetch_or(bit, std::memory_order_release);
  }
  const int rows = a.m_part ? a.m_part : a.M, cols = a.n_part ? a.n_part : a.N;
  const int tiles_m = (rows + TL::BM - 1) / TL::BM, tiles_n = (cols + TL::BN - 1) / TL::BN;  // exact without EDGE
  const int remap = (tiles_m * tiles_n) % 8 == 0 ? 1 : 0;
  // split-K (fp32 planes of partial results, forward / dgrad layouts only): a.K is the whole contraction, the kernel
  // gets the slice length and the row length of the K-contiguous operands separately
  const int slices = (EPI == E_ACCUM && AK && a.k_slices > 1) ? a.k_slices : 1;
  const dim3 grid((unsigned)(tiles_m * tiles_n), (unsigned)slices);
  kern<<<grid, TL::NT * TL::KG, lds, st>>>(a.M, a.N, a.K / slices, (const bf16_t*)a.A, (const bf16_t*)a.B, (TO*)a.C, a.bias,
                                  (const TO*)a.R, (TO*)a.C2, a.accumulate, tiles_m, remap, a.n_seg > 1 ? a.n_seg : 1,
                                  a.seg_stride_a, a.seg_stride_b, EPI == E_GELU_BWD ? a.colsum_part : nullptr, a.K);
  if (EPI == E_GELU_BWD && a.colsum_rows) *a.colsum_rows = tiles_m;
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_error("gemm_mfma launch failed: %s", hipGetErrorString(e)); return BF_EDEVICE; }
  return BF_OK;
}

template <typename TL, bool AK, bool BKC, bool EDGE>
bf_status by_epilogue(int epi, const GemmArgs& a, hipStream_t st) {
  switch (epi) {
    case E_NONE: return launch<TL, AK, BKC, E_NONE, bf16_t, EDGE>(a, st);
    case E_BIAS: return launch<TL, AK, BKC, E_BIAS, bf16_t, EDGE>(a, st);
    case E_BIAS_RES: return launch<TL, AK, BKC, E_BIAS_RES, bf16_t, EDGE>(a, st);
    case E_BIAS_GELU: return launch<TL, AK, BKC, E_BIAS_GELU, bf16_t, EDGE>(a, st);
    case E_GELU_BWD: return launch<TL, AK, BKC, E_GELU_BWD, bf16_t, EDGE>(a, st);
    default: break;
  }
  set_error("gemm_mfma: epilogue %d not available for this layout", epi);
  return BF_EINVAL;
}

template <typename TL, bool EDGE = false>
bf_status by_layout(int layout, int epi, const GemmArgs& a, hipStream_t st) {
  if constexpr (!EDGE) {
    if (epi == E_ACCUM && layout != L_TN) {  // fp32 planes of a split contraction
      if (layout == L_NN) return launch<TL, true, false, E_ACCUM, float>(a, st);
      return launch<TL, true, true, E_ACCUM, float>(a, st);
    }
  }
  if (layout == L_NN) return by_epilogue<TL, true, false, EDGE>(epi, a, st);
  if (layout == L_NT) return by_epilogue<TL, true, true, EDGE>(epi, a, st);
  if (epi != E_ACCUM) { set_error("gemm_mfma: the weight-gradient layout stores fp32 with E_ACCUM only"); return BF_EINVAL; }
  return launch<TL, false, false, E_ACCUM, float, EDGE>(a, st);
}

inline bool small_fits(int M, int N) { return M % 128 == 0 && N % 128 == 0; }
inline bool wide_fits(int layout, int epi, int M, int N) {
  if (M % 256 || N % 192) return false;
  if (layout == L_NT) return epi == E_NONE;
  return layout == L_NN && (epi == E_NONE || epi == E_BIAS || epi == E_BIAS_RES);
}
constexpr int SPLITK_TILE = 1;  // split contractions run on the 256 x 128 tile

// Tile choice: the grid runs in rounds over the chip's workgroup slots, so the estimated time of a
// tile shape is rounds x tile area / (throughput of a slot relative to a compute unit running the
// 256 x 256 tile).  Larger tiles reuse more per LDS byte; smaller ones fill the last round.  A
// partly filled last round counts as (1 + fill) / 2 of a round: the chip runs at its power limit,
// and the compute units that do work clock higher when the others idle (measured: 384 large tiles
// beat 768 of 256 x 128, 128 large tiles lose to 256 of them).
// 0: 256 x 256 (one per compute unit), 1: 256 x 128 (one), 2: 128 x 128 (two), 3: 256 x 192 (one; only where the
// caller says the product can take it).
// est: where the estimate goes (in outputs of a 256 x 256 tile per compute unit).
inline int choose_tile(int M, int N, bool wide = false, double* est = nullptr) {
  const int bm[4] = {256, 256, 128, 256}, bn[4] = {256, 128, 128, 192};
  const long slots[4] = {256, 256, 512, 256};
  const double rate[4] = {1.0, TILE_RATE_MID, TILE_RATE_SMALL / 2, TILE_RATE_WIDE};
  int best = -1;
  double best_t = 0;
  for (int i = 0; i < (wide ? 4 : 3); ++i) {
    if (M % bm[i] || N % bn[i]) continue;
    const long tiles = (long)(M / bm[i]) * (N / bn[i]), full = tiles / slots[i], rest = tiles % slots[i];
    const double rounds = (double)full + (rest ? 0.5 + 0.5 * (double)rest / slots[i] : 0.0);
    const double t = rounds * bm[i] * bn[i] / rate[i];
    if (best < 0 || t < best_t) { best = i; best_t = t; }
  }
  if (est) *est = best_t;
  return best;
}

// Time of a k-tile (64 of K) on 256 x 256 tiles with every compute unit at work, and of starting another kernel, us.
constexpr double K_TILE_US = 1.65, LAUNCH_US = 3.0;

// Products of few tiles run on 64 x 64 ones, whole or not: a workgroup that has a compute unit to itself takes 1.2, 0.72,
// 0.6-0.7 and 0.3 us per k-tile on 256 x 256, 256 x 128, 128 x 128 and 64 x 64 (two of the last: 0.5), so up to two of
// them per compute unit the smallest tile is the fastest.  Measured (forward / dgrad layout, the best whole tile
// against 64 x 64): 128 x 1024 x 1024 12.3 / 7.2 us, 1024 x 1024 x 2048 24.4 / 12.9, 1024 x 2048 x 2048 24.9 / 17.9; 1024 x
// 3072 x 1024 (768 tiles) 14.3 / 14.0, 2048 x 2048 x 2048 (1024) 25.6 / 27.7.  Weight-gradient layout, whose transpose
// loads make more of the smaller tile: 1024 x 1024 x 2048 (256 tiles) 21.3 / 16.7, 1024 x 2048 x 2048 (512) 22.4 / 23.0.
inline bool few_tiles(int layout, int M, int N) {
  return (long)((M + 63) / 64) * ((N + 63) / 64) <= (layout == L_TN ? 256 : 512);
}

// Few tiles and a contraction of some length: a tile's k-tiles are a chain of loads, barriers and fragment reads that one
// or two workgroups per compute unit do not overlap, so two (or four) groups of waves share it, each on every second
// (fourth) k-tile with LDS stages of its own, and add their sums in LDS at the end.  More than 256 tiles of 64 x 64 (two
// workgroups to a unit already) also take 128 x 64 ones, which load a quarter less per product.  One group / two / four on 64 x 64 / two on
// 128 x 64, us: forward 1000 x 2048 x 8192 75.0 / 67.2 / - / 53.0, dgrad 59.4 / 53.3 / - / 46.2, forward 1000 x 2048 x 2048 18.8 / 17.3 / - / 16.5,
// dgrad 1100 x 1000 x 1024 9.2 / 9.1 / 11.9 / 8.7; forward 1000 x 1024 x 8192 55.3 / 37.8 / 33.1 / 46.1, 500 x 1024 x 4096 31.7 / 20.6 / 17.3 /
// 25.7, 300 x 512 x 2048 12.9 / 10.7 / 10.3 / 14.4, 64 x 512 x 50304 350 / 207 / 153 / 252, dgrad 128 x 256 x 1024 6.7 / 6.0 / 6.4 / 8.1, 1000 x 1000 x 768 7.5 /
// 7.2 / 7.9 / 8.9.  Weight gradients, one / two on 64 x 64: 512 x 512 over 4096 28.4 / 20.6, 1024 x 1024 over 1000 9.6 / 8.0, 512 x 512 over 512 5.9 / 5.4,
// 1000 x 1024 over 300 5.4 / 5.5.  (Four groups there want more LDS than there is.)
enum Groups { G_ONE, G_TWO, G_FOUR, G_TWO_TALL };
inline Groups key_groups(int layout, int M, int N, int K, int n_seg) {
  if (!few_tiles(layout, M, N) || n_seg > 1) return G_ONE;
  if (layout == L_TN) return K >= 512 ? G_TWO : G_ONE;
  if (K < 1024) return G_ONE;
  if ((long)((M + 63) / 64) * ((N + 63) / 64) > 256) return G_TWO_TALL;
  return K >= 4096 ? G_FOUR : G_TWO;
}

// Tile of the edge form: 0: 256 x 256, 1: 128 x 128 (by the estimate of choose_tile, the last tiles partly empty), 2: 64 x 64.
inline int choose_edge_tile(int layout, int M, int N) {
  if (few_tiles(layout, M, N)) return 2;
  const int e[2] = {256, 128};
  const long slots[2] = {256, 512};
  const double rate[2] = {1.0, TILE_RATE_SMALL / 2};
  double t[2];
  for (int i = 0; i < 2; ++i) {
    const long tiles = (long)((M + e[i] - 1) / e[i]) * ((N + e[i] - 1) / e[i]), full = tiles / slots[i], rest = tiles % slots[i];
    t[i] = ((double)full + (rest ? 0.5 + 0.5 * (double)rest / slots[i] : 0.0)) * e[i] * e[i] / rate[i];
  }
  return t[0] < t[1] ? 0 : 1;
}

}  // namespace

bool gemm_mfma_edge_supported(int layout, int epi, int M, int N, int K) {
  if (layout < L_NN || layout > L_TN || (layout == L_TN) != (epi == E_ACCUM) || epi < E_NONE || epi > E_ACCUM) return false;
  if (M < 1 || N < 1 || K < 1 || N % 8) return false;
  const long ldmax = 1l << 21;  // 32-bit lane offsets over 256 rows (K is a row's length, but for the weight gradient)
  if (M > ldmax || N > ldmax || (layout != L_TN && K > ldmax)) return false;
  return layout == L_TN ? M % 8 == 0 : K % 8 == 0;
}

bool gemm_mfma_few_tiles(int layout, int M, int N) { return few_tiles(layout, M, N); }

// Weight gradients of odd multiples of 128 (a 50304-word vocabulary: 393 x 128) on 256 x 256 tiles whose last row is half
// empty: 50304 x 2048 over 2048 tokens 603 -> 451 us.  The other layouts have the 256 x 192 and 256 x 128 tiles there.
bool gemm_mfma_edge_better(int layout, int M, int N) {
  if (few_tiles(layout, M, N)) return true;
  if (layout != L_TN || !(M % 256 || N % 256) || choose_tile(M, N) != 2) return false;
  return choose_edge_tile(layout, M, N) == 0;
}

bf_status gemm_mfma_edge(int layout, int epi, const GemmArgs& a, hipStream_t st) {
  if (!gemm_mfma_edge_supported(layout, epi, a.M, a.N, a.K)) { set_error("gemm_mfma: shape not supported"); return BF_EINVAL; }
  if (a.n_seg > 1 && (layout != L_TN || ((a.seg_stride_a | a.seg_stride_b) & 7))) {
    set_error("gemm_mfma: segments go with the weight-gradient layout and 16-byte aligned strides");
    return BF_EINVAL;
  }
  const uintptr_t al = (uintptr_t)a.A | (uintptr_t)a.B | (uintptr_t)a.C | (uintptr_t)a.R | (uintptr_t)a.C2 | (uintptr_t)a.bias;
  if (al & 15) { set_error("gemm_mfma: operands must be 16-byte aligned"); return BF_EINVAL; }
  switch (choose_edge_tile(layout, a.M, a.N)) {
    case 0: return by_layout<TileBig, true>(layout, epi, a, st);
    case 1: return by_layout<TileSmall, true>(layout, epi, a, st);
    default: break;
  }
  GemmArgs b = a;
  if (a.n_seg > 1 && a.seg_stride_a == (size_t)a.K * a.M && a.seg_stride_b == (size_t)a.K * a.N && (long)a.K * a.n_seg < (1l << 31)) {
    // segments that follow each other without a gap are one contraction
    b.K = a.K * a.n_seg;
    b.n_seg = 1;
  }
  switch (key_groups(layout, b.M, b.N, b.K, b.n_seg)) {
    case G_TWO: return by_layout<TileTiny2, true>(layout, epi, b, st);
    case G_FOUR: return layout == L_NN ? by_epilogue<TileTiny4, true, false, true>(epi, b, st) : by_epilogue<TileTiny4, true, true, true>(epi, b, st);
    case G_TWO_TALL: return layout == L_NN ? by_epilogue<TileTall2, true, false, true>(epi, b, st) : by_epilogue<TileTall2, true, true, true>(epi, b, st);
    default: return by_layout<TileTiny, true>(layout, epi, b, st);
  }
}

bool gemm_mfma_supported(int layout, int epi, int M, int N, int K) {
  if (layout < L_NN || layout > L_TN) return false;
  if ((layout == L_TN) != (epi == E_ACCUM)) return false;
  if (epi < E_NONE || epi > E_ACCUM) return false;
  if (M < 1 || N < 1 || K < BK || K % BK) return false;
  return small_fits(M, N);
}

void gemm_mfma_tile(int layout, int epi, int M, int N, int* bm, int* bn) {
  const int rows[4] = {256, 256, 128, 256}, cols[4] = {256, 128, 128, 192};
  const int t = choose_tile(M, N, wide_fits(layout, epi, M, N));
  *bm = t < 0 ? 0 : rows[t];
  *bn = t < 0 ? 0 : cols[t];
}

// Whole rounds and a rest.  A grid of 256 x 256 tiles that fills the chip several times over and then a few tiles' width
// more (50304 columns by 2048 rows: 6.14 rounds, and 50304 is no multiple of 256) runs the whole rounds by themselves and the
// rest, whole tiles of 128, as a second launch on the tile that suits it, where the estimates of the two and a launch come to less
// than that of one grid.  Rows of the weight gradient (M), columns of the others.  One grid / two, us: dgrad layout 2048 x
// 50304 x 2048 393 / 365 (256 x 192 tiles), x 512 138 / 130, 1024 x 50304 x 1024 115 / 108, 2048 x 8320 x 2048 89 / 79; forward 431 / 409; weight gradient
// 50304 x 2048 x 2048 436 / 393, 50304 x 1024 x 2048 236 / 212, 9216 x 2048 x 4096 187 / 147; not taken: 50304 x 512 x 2048 116 / 126, dgrad 2048 x
// 9216 x 8192 270 / 278 (1.5 rounds of 256 x 192), 2048 x 32000 x 1024 123 / 126.
// Sizes whose 256-wide tiles across do not divide 256 (1536, 3072, 6144) keep one grid: a round of theirs is no rectangle.
// 0, or the rows / columns of the whole rounds.
static int whole_rounds(int layout, int epi, int M, int N, int K, bool shared_chip) {
  const int fixed = layout == L_TN ? N : M, var = layout == L_TN ? M : N, across = fixed / 256;
  if (fixed % 256 || across > 256 || 256 % across) return 0;
  const int unit = 256 / across * 256, main = var / unit * unit, rest = var - main;
  if (!main || !rest || rest % 128) return 0;
  double one, two;
  if (layout == L_TN && choose_edge_tile(layout, M, N) == 0) {
    const long tiles = (long)((M + 255) / 256) * (N / 256), last = tiles % 256;
    one = ((double)(tiles / 256) + (last ? 0.5 + 0.5 * (double)last / 256 : 0.0)) * 65536;
  } else {
    choose_tile(M, N, !shared_chip && wide_fits(layout, epi, M, N), &one);
  }
  choose_tile(layout == L_TN ? rest : M, layout == L_TN ? N : rest, false, &two);
  two += (double)main / unit * 65536;
  const double us = (double)K / BK * K_TILE_US / 65536;
  return two * us + LAUNCH_US < one * us ? main : 0;
}

bool gemm_mfma_in_rounds(int layout, int epi, const GemmArgs& a) {
  // (partial column sums have a row per row of tiles of the one grid)
  return a.n_seg <= 1 && !(epi == E_GELU_BWD && a.colsum_part) && !few_tiles(layout, a.M, a.N) && whole_rounds(layout, epi, a.M, a.N, a.K, a.shared_chip) > 0;
}

static bf_status in_rounds(int layout, int epi, const GemmArgs& a, int main, hipStream_t st) {
  GemmArgs b = a;
  (layout == L_TN ? b.m_part : b.n_part) = main;
  bf_status r = by_layout<TileBig>(layout, epi, b, st);
  if (r != BF_OK) return r;
  // the rest: the same matrices from row / column `main` on
  b = a;
  const size_t m = (size_t)main;
  if (layout == L_TN) {
    b.A = (const bf16_t*)a.A + m;
    b.C = (float*)a.C + m * a.N;
    b.m_part = a.M - main;
  } else {
    b.B = (const bf16_t*)a.B + (layout == L_NT ? m * a.K : m);
    b.C = (bf16_t*)a.C + m;
    if (a.bias) b.bias = a.bias + m;
    if (a.R) b.R = (const bf16_t*)a.R + m;
    if (a.C2) b.C2 = (bf16_t*)a.C2 + m;
    b.n_part = a.N - main;
  }
  switch (layout == L_TN ? choose_tile(a.M - main, a.N) : choose_tile(a.M, a.N - main)) {
    case 0: return by_layout<TileBig>(layout, epi, b, st);
    case 1: return by_layout<TileMid>(layout, epi, b, st);
    default: return by_layout<TileSmall>(layout, epi, b, st);
  }
}

// Slices of a very long contraction (a 50304-word vocabulary's) on 256 x 256 tiles, as many as make the estimate of rounds and
// of the pass over the planes the least; 0: not for these.  256 x 128 tiles in two slices / here, us: 2048 x 2048 x 50304 416 / 400 (3), 2048 x
// 1024 x 50304 360 / 217 (6), 1024 x 1536 x 50304 314 / 189 (6), 2048 x 1024 x 32000 201 / 163 (4); at K = 8192 level (2048 x 2048 75.7 / 76.6 in 4, 1024 x
// 2048 58.0 / 55.9), where two planes are less scratch.  Up to 256 tiles of 64 x 64 two slices run on those, at 0.4 us per 128 of K
// against 1.2 us per 64 of K and slice here: from six slices on.  Two on 64 x 64 / here: 256 x 1024 x 16384 55.5 / 48.5 (8), 512 x 512 x
// 50304 161 / 160 (6; dgrad layout, 256 rows 157 / 159), 512 x 2048 x 50304 219 / 170, but 256 x 1024 x 32000 101 / 124 (5), 1024 x 1024 x 32000 116 / 128.
static int big_slices(int M, int N, int K) {
  if (K < 16384 || M % 256 || N % 256 || K % BK) return 0;
  const long tiles = (long)(M / 256) * (N / 256);
  if (tiles > 128) return 0;
  int best = 0;
  double best_t = 0;
  for (int s = 2; s <= 8; ++s) {
    if (K % (s * BK)) continue;
    const long wgs = tiles * s, last = wgs % 256;
    const double rounds = (double)(wgs / 256) + (last ? 0.5 + 0.5 * (double)last / 256 : 0.0);
    const double t = rounds * (K / s / BK) * K_TILE_US + s * (double)M * N * 8 / 4.5e6;  // planes written and read at 4.5 TB/s
    if (!best || t < best_t) { best = s; best_t = t; }
  }
  return best < 6 && (M / 64) * (N / 64) <= 256 ? 0 : best;
}

bf_status gemm_mfma(int layout, int epi, const GemmArgs& a, hipStream_t st) {
  const bool planes = epi == E_ACCUM && layout != L_TN;  // split contraction of a forward / dgrad product
  if (planes) {
    if (a.k_slices < 2 || a.K % (a.k_slices * BK) || !gemm_mfma_supported(layout, E_NONE, a.M, a.N, a.K / a.k_slices) || a.accumulate ||
        a.n_seg > 1) {
      set_error("gemm_mfma: bad split of the contraction (%d slices of K = %d)", a.k_slices, a.K);
      return BF_EINVAL;
    }
  } else if (!gemm_mfma_supported(layout, epi, a.M, a.N, a.K)) { set_error("gemm_mfma: shape not supported"); return BF_EINVAL; }
  if (a.n_seg > 1 && (layout != L_TN || ((a.seg_stride_a | a.seg_stride_b) & 7))) {
    set_error("gemm_mfma: segments go with the weight-gradient layout and 16-byte aligned strides");
    return BF_EINVAL;
  }
  const uintptr_t al = (uintptr_t)a.A | (uintptr_t)a.B | (uintptr_t)a.C | (uintptr_t)a.R | (uintptr_t)a.C2 | (uintptr_t)a.bias;
  if (al & 15) { set_error("gemm_mfma: operands must be 16-byte aligned"); return BF_EINVAL; }
  if (planes && a.k_slices == big_slices(a.M, a.N, a.K))
    return layout == L_NN ? launch<TileBig, true, false, E_ACCUM, float>(a, st) : launch<TileBig, true, true, E_ACCUM, float>(a, st);
  // slices of a product of few tiles: on 64 x 64 as well, as long as both slices' workgroups find room
  if (planes && (long)(a.M / 64) * (a.N / 64) <= 256)
    return layout == L_NN ? launch<TileTiny, true, false, E_ACCUM, float>(a, st) : launch<TileTiny, true, true, E_ACCUM, float>(a, st);
  if (!planes && gemm_mfma_in_rounds(layout, epi, a)) return in_rounds(layout, epi, a, whole_rounds(layout, epi, a.M, a.N, a.K, a.shared_chip), st);
  switch (planes ? SPLITK_TILE : choose_tile(a.M, a.N, !a.shared_chip && wide_fits(layout, epi, a.M, a.N))) {
    case 0: return by_layout<TileBig>(layout, epi, a, st);
    case 1: return by_layout<TileMid>(layout, epi, a, st);
    case 3:
      if (layout == L_NT) return launch<TileWide, true, true, E_NONE, bf16_t>(a, st);
      if (epi == E_BIAS) return launch<TileWide, true, false, E_BIAS, bf16_t>(a, st);
      if (epi == E_BIAS_RES) return launch<TileWide, true, false, E_BIAS_RES, bf16_t>(a, st);
      return launch<TileWide, true, false, E_NONE, bf16_t>(a, st);
    default: return by_layout<TileSmall>(layout, epi, a, st);
  }
}

// Split-K.  A product whose best tile shape still leaves half of the workgroup slots of its only round empty (the
// 2048-column products of a 2048-wide model on 2048-row micro-batches: 128 tiles of 256 x 128) runs its contraction
// in two slices on twice as many workgroups; each slice leaves an fp32 plane and a second kernel adds the planes in
// ascending order and applies the epilogue, so the result does not depend on which slice finishes first.  Measured on
// the step of a 2048-wide, 6-layer model (8 micro-batches of 2048 rows): 48.8 -> 44.6 ms with K >= 4096 split, 44.3 with
// K >= 2048; four slices on 256 x 256 tiles instead: 45.6.
// Products of few tiles (64 x 64 ones) fill the chip better unsplit, and the second pass only pays for a longer contraction:
// a k-tile takes 0.31 us on up to 256 of those and 0.47 on twice as many, so two slices save a quarter of the loop
// and cost a pass over the planes (6 us).  1024 x 1024 x 8192: 55 us unsplit, 38 split (55 in slices of 256 x 128 tiles);
// 1024 x 2048 x 4608: 40 either way; 1024 x 1024 x 2048: 13 against 14 and more.
constexpr int SPLITK_FEW_TILES_K = 4608;

// fits: planes that the caller has room for
int gemm_splitk_slices(int layout, int epi, int M, int N, int K, int fits) {
  if (layout != L_NN && layout != L_NT) return 1;
  if (epi != E_NONE && epi != E_BIAS && epi != E_BIAS_RES) return 1;
  if (K < 2048 || K % (2 * BK) || !gemm_mfma_supported(layout, epi, M, N, K)) return 1;
  if (M % 256 || N % 128) return 1;
  const int big = big_slices(M, N, K);
  if (big && big <= fits) return big;
  if (fits < 2) return 1;
  if (K < SPLITK_FEW_TILES_K && few_tiles(layout, M, N)) return 1;
  if (choose_tile(M, N) != SPLITK_TILE) return 1;
  const long tiles = (long)(M / 256) * (N / 128);
  return tiles <= 128 ? 2 : 1;
}

}  // namespace bf
