// GEMM on the gfx950 matrix cores in full fp32 (v_mfma_f32_32x32x2_f32 / 16x16x4_f32: fp32 operands, fp32 accumulate),
// any shape, all three operand layouts and all epilogues.  It is the fp32-mode product, and takes the bf16 products whose
// rows are not whole 16-byte chunks (the operands are widened on their way into LDS).
//
// The instructions round after every product, in the order of their k, so a product contracted in ascending k is the
// chain of fused multiply-adds the vector kernel (gemm_plain.hip) computes: the same bits, which the tests check.  That is
// why no tile splits the contraction and why a stage-wide weight gradient keeps one chain per segment.
//
// They contract at 64 flop per clock and SIMD (157 TFLOP/s over the chip), so an LDS float feeds enough work that only the
// matrix pipeline and what the waves issue beside it count: one barrier per k-tile, global -> registers -> LDS with two
// tiles in flight in registers, a few scalar instructions per tile (the waves of a compute unit share one scalar unit:
// recomputing addresses for every tile held the 128 x 128 tile at 117 TFLOP/s, advancing them gives 136 at 8192^3; the
// installed library 154), and everything else of a k-tile issued behind an MFMA (see the loop).  Products of an fp32 layer of
// width 1024 on 512 tokens, vector kernel / this one with the rest of a k-tile in one piece and an epilogue that waits for each
// of its reads / now: 1024 -> 4096 220 / 56 / 49 us, 4096 -> 1024 842 / 58 / 55, weight gradient 139 / 54 / 46, the whole
// MLP 306 -> 271; a plain 1024 x 4096 output 116 -> 124 TFLOP/s at K = 1024 and 124 -> 135 at 4096, transposed operands 98 -> 117.  What is
// left at 512 x 1024 x 4096: two waves per SIMD of one 16 x 16 accumulator each (a 64 x 32 tile of two chains per wave: the same
// 49 us), rows 16 KB apart in one tile.
#include <type_traits>

#include "common.h"
#include "epilogue.h"

namespace bf {

namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

constexpr int NT = 256;

// WM x WN waves side by side, each owning MI x NI MFMA tiles of MT x MT (v_mfma_f32_32x32x2 or 16x16x4)
template <int WM_, int WN_, int MI_, int NI_, int BK_, int MT_>
struct Cfg {
  static constexpr int WM = WM_, WN = WN_, MI = MI_, NI = NI_, BK = BK_, MT = MT_;
  static constexpr int BM = WM * MI * MT, BN = WN * NI * MT;
  static constexpr int KG = MT == 32 ? 8 : 16;  // k that four MFMA steps contract
  static constexpr int KW = BK / KG;
  static constexpr int NR = MT == 32 ? 16 : 4;  // accumulator registers per tile
  static_assert(WM * WN == NT / 64 && KW >= 1, "four waves");
};

// ---- global -> registers -> LDS: VEC adjacent elements per access, widened to fp32.  The descriptor of the buffer loads
// ends where the matrix (or the segment of a stage-wide weight gradient) ends: rows past the matrix read as zero, and
// so does what lies past K (sent past the end where K is the fast dimension).  Elements past the other extent of a
// K-slow operand belong to its next row and only reach outputs that are not stored.
// MT = 32: lane l's k of step s is 2 s + l / 32; a K-contiguous row is laid down with the even k of every group of 8 in
// front of the odd ones, so that a lane's four steps are one 16-byte read.  MT = 16: k = 4 s + l / 16, 4-byte reads.
template <typename TI, int VEC, bool KCONTIG, int R, int BK, int MT>
struct Stage {
  // row pitches at which the fragment reads are conflict-free
  static constexpr int LD = KCONTIG ? BK + 4 : MT == 32 ? R + 32 : R + 16;
  static constexpr int ELEMS = KCONTIG ? R * LD : BK * LD;
  static constexpr int CPR = (KCONTIG ? BK : R) / VEC;  // chunks per row of the tile as it lies in memory
  static constexpr int STEP = NT / CPR;                 // rows between a thread's chunks
  static constexpr int CHUNKS = (KCONTIG ? R : BK) / STEP;
  static_assert(NT % CPR == 0 && (KCONTIG ? R : BK) % STEP == 0, "the tile's chunks must divide among the threads");
  // Where the operand's next tile starts and what is left of the matrix from there (elements): advanced tile by tile, so
  // that a k-tile costs a handful of scalar instructions (all waves of a compute unit share one scalar unit).
  struct Walk {
    const TI* p;
    long left, per_tile, left0;
    __device__ __forceinline__ void init(const TI* g, size_t ld, int r0, int R_ext, int K) {
      p = KCONTIG ? g + (size_t)r0 * ld : g + r0;
      left0 = left = KCONTIG ? (long)(R_ext - r0) * (long)ld : (long)K * (long)ld - r0;
      per_tile = KCONTIG ? BK : BK * (long)ld;
    }
    __device__ __forceinline__ void next() { p += per_tile; left -= per_tile; }
  };
  typename std::conditional<VEC == 4, f32x4, float>::type v[CHUNKS];
  uint32_t goff, step;
  int loff, kcol;
  __device__ __forceinline__ void init(size_t ld, int tid) {
    const int row = tid / CPR, c = (tid % CPR) * VEC;
    goff = (uint32_t)(((size_t)row * ld + c) * sizeof(TI));
    step = (uint32_t)((size_t)STEP * ld * sizeof(TI));
    loff = row * LD + (KCONTIG && MT == 32 ? (c & ~7) + ((c & 1) << 2) + ((c & 7) >> 1) : c);
    kcol = c;
  }
  // k_left: k from the tile's start to the end (not positive past the last tile: the loop's loads have no branch around
  // them, which would make the compiler wait for all of them at once; they return zeros without touching memory)
  __amdgpu_buffer_rsrc_t rsrc;
  uint32_t off;
  __device__ __forceinline__ void aim(const Walk& wk, int k_left) {
    const long cap = (long)(0x7fffff00 / sizeof(TI));
    const long n = wk.left < cap ? (wk.left > 0 ? wk.left : 0) : cap;
    rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)wk.p, 0, (int)(n * (long)sizeof(TI)), 0x00020000);
    off = KCONTIG && kcol >= k_left ? 0x7fffff00u : goff;
  }
  __device__ __forceinline__ void load(int i) {
    if constexpr (VEC == 4) {
      static_assert(std::is_same<TI, float>::value, "wide chunks are fp32");
      v[i] = __builtin_bit_cast(f32x4, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(rsrc, off + i * step, 0, 0));
    } else if constexpr (std::is_same<TI, float>::value) {
      v[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, off + i * step, 0, 0));
    } else {
      v[i] = __builtin_bit_cast(float, (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rsrc, off + i * step, 0, 0) << 16);
    }
  }
  __device__ __forceinline__ void store(float* lds, int i) const {
    float* d = lds + loff + i * STEP * LD;
    if constexpr (VEC == 4 && KCONTIG && MT == 32) {
      *reinterpret_cast<f32x2*>(d) = f32x2{v[i][0], v[i][2]};
      *reinterpret_cast<f32x2*>(d + 4) = f32x2{v[i][1], v[i][3]};
    } else if constexpr (VEC == 4) {
      *reinterpret_cast<f32x4*>(d) = v[i];
    } else {
      *d = v[i];
    }
  }
  // values of the four MFMA steps of k group kg for row / column r0 + lane % MT
  static __device__ __forceinline__ f32x4 frag(const float* lds, int r0, int kg, int lane) {
    const int r = r0 + (lane & (MT - 1)), q = lane / MT;
    if constexpr (KCONTIG && MT == 32) {
      return *reinterpret_cast<const f32x4*>(lds + r * LD + kg * 8 + 4 * q);
    } else {
      constexpr int KS = MT == 32 ? 2 : 4;  // k per step
      f32x4 o;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int k = (kg * 4 + t) * KS + q;
        o[t] = KCONTIG ? lds[r * LD + k] : lds[k * LD + r];
      }
      return o;
    }
  }
};

template <int MT>
struct Acc;
template <>
struct Acc<32> {
  typedef f32x16 T;
  static __device__ __forceinline__ T mma(float a, float b, T c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
  static __device__ __forceinline__ int row(int r, int lane) { return (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3); }
};
template <>
struct Acc<16> {
  typedef f32x4 T;
  static __device__ __forceinline__ T mma(float a, float b, T c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  static __device__ __forceinline__ int row(int r, int lane) { return (lane >> 4) * 4 + r; }
};

// A wave's elements of a row-major M x N matrix, in the order of its accumulators.  The descriptor ends where the matrix does and
// columns past N are sent past its end: nothing is read or written there, and there is no branch around an access.
template <typename C, typename TO>
struct Outer {
  __amdgpu_buffer_rsrc_t rsrc;
  int col0, N;
  uint32_t base, pitch;
  __device__ __forceinline__ Outer(TO* p, int m0, int n0, int M, int N_, int wm, int wn, int lane) {
    const long left = (long)(M - m0) * N_ * (long)sizeof(TO);
    rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(p + (size_t)m0 * N_), 0, (int)(left < 0x7fffff00 ? left : 0x7fffff00), 0x00020000);
    N = N_;
    col0 = n0 + wn * C::NI * C::MT + (lane & (C::MT - 1));
    pitch = (uint32_t)N_ * sizeof(TO);
    base = (uint32_t)(wm * C::MI * C::MT + Acc<C::MT>::row(0, lane)) * pitch + (uint32_t)col0 * sizeof(TO);
  }
  __device__ __forceinline__ uint32_t off(int i, int j, int r) const {
    return col0 + j * C::MT < N ? base + (uint32_t)(i * C::MT + Acc<C::MT>::row(r, 0)) * pitch + j * C::MT * (uint32_t)sizeof(TO) : 0x7fffff00u;
  }
  __device__ __forceinline__ float load(int i, int j, int r) const {
    if constexpr (std::is_same<TO, float>::value) return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, off(i, j, r), 0, 0));
    else return __builtin_bit_cast(float, (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rsrc, off(i, j, r), 0, 0) << 16);
  }
  __device__ __forceinline__ void store(TO v, int i, int j, int r) const {
    if constexpr (std::is_same<TO, float>::value) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), rsrc, off(i, j, r), 0, 0);
    else __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, v), rsrc, off(i, j, r), 0, 0);
  }
};

// one tile of a product
template <typename C, typename TI, int VEC, bool AK, bool BKC, int EPI, typename TO>
__device__ __forceinline__ void tile_product(int lin, int M, int N, int K, const TI* __restrict__ A, const TI* __restrict__ B, TO* __restrict__ Cm,
                                             const float* __restrict__ bias, const TO* __restrict__ R, TO* __restrict__ C2, int accumulate,
                                             int tiles_m, int n_seg, size_t seg_a, size_t seg_b) {
  typedef Stage<TI, VEC, AK, C::BM, C::BK, C::MT> SA;
  typedef Stage<TI, VEC, BKC, C::BN, C::BK, C::MT> SB;
  typedef Acc<C::MT> AC;
  constexpr int STAGE = SA::ELEMS + SB::ELEMS;
  __shared__ __attribute__((aligned(16))) float smem[2 * STAGE];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int wm = w % C::WM, wn = w / C::WM;
  const int m0 = lin % tiles_m * C::BM, n0 = lin / tiles_m * C::BN;
  const size_t lda = AK ? K : M, ldb = BKC ? K : N;
  // Sums of one segment; of all segments so far (weight gradients: one chain per micro-batch, added in order to what the
  // main-grad holds, as one product per micro-batch would)
  typename AC::T acc[C::MI][C::NI], tot[C::MI][C::NI];
  auto each = [&](auto f) {
#pragma unroll
    for (int i = 0; i < C::MI; ++i)
#pragma unroll
      for (int j = 0; j < C::NI; ++j)
#pragma unroll
        for (int r = 0; r < C::NR; ++r) f(i, j, r);
  };
  // What the epilogue reads.  Element by element between the stores every read waits for the memory by itself, 10 us of a
  // product's 57 at 512 x 1024 x 4096; so all are requested together, in front of the k loop where their registers cost
  // no second workgroup on the compute unit.
  constexpr bool READS_R = EPI == E_BIAS_RES || EPI == E_GELU_BWD, EARLY_R = C::MI * C::NI <= 2;
  typedef Outer<C, TO> OT;
  const OT out(Cm, m0, n0, M, N, wm, wn, lane), out2(EPI == E_BIAS_GELU ? C2 : Cm, m0, n0, M, N, wm, wn, lane);
  typename AC::T rv[C::MI][C::NI];
  float bv[C::NI];
  auto read_r = [&] {
    const OT from((TO*)R, m0, n0, M, N, wm, wn, lane);
    each([&](int i, int j, int r) { rv[i][j][r] = from.load(i, j, r); });
  };
  auto read_ahead = [&] {
    each([&](int i, int j, int r) {
      acc[i][j][r] = 0.f;
      tot[i][j][r] = 0.f;
    });
    if constexpr (EPI == E_ACCUM)
      if (accumulate) each([&](int i, int j, int r) { tot[i][j][r] = out.load(i, j, r); });
#pragma unroll
    for (int j = 0; j < C::NI; ++j) bv[j] = EPI == E_BIAS || EPI == E_BIAS_RES || EPI == E_BIAS_GELU ? bias[min(out.col0 + j * C::MT, N - 1)] : 0.f;
    if constexpr (READS_R && EARLY_R) read_r();
  };
  SA sa[2];  // set t & 1 carries tile t
  SB sb[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    sa[q].init(lda, tid);
    sb[q].init(ldb, tid);
  }
  const int nk_seg = (K + C::BK - 1) / C::BK, nk = nk_seg * n_seg;
  typename SA::Walk wa;
  typename SB::Walk wb;
  wa.init(A, lda, m0, M, K);
  wb.init(B, ldb, n0, N, K);
  int k_left = K, seg = 0;
  typedef std::integral_constant<int, 0> I0;
  typedef std::integral_constant<int, 1> I1;
  constexpr int NCA = SA::CHUNKS, NC = SA::CHUNKS + SB::CHUNKS;
  auto aim = [&](auto setc) {
    constexpr int SET = decltype(setc)::value;
    sa[SET].aim(wa, k_left);
    sb[SET].aim(wb, k_left);
    wa.next();
    wb.next();
    k_left -= C::BK;
    if (EPI == E_ACCUM && k_left <= 0) {  // the next segment, or nothing more
      ++seg;
      k_left = K;
      wa.p = A + (size_t)seg * seg_a + m0;
      wb.p = B + (size_t)seg * seg_b + n0;
      wa.left = seg < n_seg ? wa.left0 : 0;
      wb.left = seg < n_seg ? wb.left0 : 0;
    }
  };
  auto load = [&](auto setc, int c) {
    constexpr int SET = decltype(setc)::value;
    if (c < NCA) sa[SET].load(c);
    else sb[SET].load(c - NCA);
  };
  auto store = [&](auto setc, int stage, int c) {
    constexpr int SET = decltype(setc)::value;
    if (c < NCA) sa[SET].store(smem + stage * STAGE, c);
    else sb[SET].store(smem + stage * STAGE + SA::ELEMS, c - NCA);
  };
  // fragments of the k group being contracted and of the next one
  constexpr int NF = C::MI + C::NI;
  f32x4 a[2][C::MI], b[2][C::NI];
  auto fetch = [&](int buf, int stage, int g, int f) {
    const float* as = smem + stage * STAGE;
    if (f < C::MI) a[buf][f] = SA::frag(as, (wm * C::MI + f) * C::MT, g, lane);
    else b[buf][f - C::MI] = SB::frag(as + SA::ELEMS, (wn * C::NI + f - C::MI) * C::MT, g, lane);
  };
  // Tiles are requested three iterations before they are contracted (two register sets and an LDS stage).  One barrier per
  // k-tile, in its last group: by then every wave holds that group's fragments in registers and has written
  // tile kt + 1 into the other stage, so the first fragments of the next tile arrive under the rest of the group's MFMAs.
  // A wave is alone on its SIMD or shares it with one more and issues in order, so whatever stands between two groups
  // leaves the matrix pipeline idle: the next group's fragments, the stores of the next tile and the loads of the
  // one after go one or two at a time behind an MFMA each (64 cycles, of which its issue takes four).  Not so the stores and
  // loads of the smallest tile with K-contiguous rows: its k-tile is 16 short MFMAs, and loads a third of it later are not back
  // in time for long contractions.  In front of the first MFMA / behind them, us: 768 x 256 x 2048 dgrad layout 16.6 / 17.7, forward
  // 16.6 / 17.3, x 4096 30.4 / 32.3, 30.2 / 31.7, x 1024 level; weight gradient, whose rows are short, x 2048 21.6 / 17.1.
  constexpr bool FRONT = C::MT == 16 && AK;
  constexpr int NG = 4 * C::MI * C::NI, PRE = NG / 4;                    // MFMAs of a group; those in front of the barrier
  constexpr int PER = (2 * NC + (C::KW - 1) * (NG - NF) - 1) / ((C::KW - 1) * (NG - NF));  // stores and loads behind one MFMA
  auto iter = [&](auto stagec) {
    constexpr int CUR = decltype(stagec)::value;  // LDS stage
    typedef std::integral_constant<int, CUR ^ 1> Next;
    if constexpr (FRONT) {
#pragma unroll
      for (int c = 0; c < NC; ++c) store(Next{}, CUR ^ 1, c);
      aim(Next{});
#pragma unroll
      for (int c = 0; c < NC; ++c) load(Next{}, c);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int g = 0; g < C::KW; ++g) {
      const int buf = g & 1;
#pragma unroll
      for (int m = 0; m < NG; ++m) {
        const int s = m / (C::MI * C::NI), i = m / C::NI % C::MI, j = m % C::NI;
        acc[i][j] = AC::mma(a[buf][i][s], b[buf][j][s], acc[i][j]);
        if (g + 1 < C::KW) {
          if (m < NF) {
            fetch(buf ^ 1, CUR, g + 1, m);
          } else if constexpr (!FRONT) {
#pragma unroll
            for (int q = 0; q < PER; ++q) {
              const int item = (g * (NG - NF) + m - NF) * PER + q;
              if (item < NC) store(Next{}, CUR ^ 1, item);
              if (item == NC) aim(Next{});
              if (item >= NC && item < 2 * NC) load(Next{}, item - NC);
            }
          }
        } else if (m == PRE - 1) {
          __builtin_amdgcn_sched_barrier(0);
          __syncthreads();
#pragma unroll
          for (int f = 0; f < NF; ++f) fetch(buf ^ 1, CUR ^ 1, 0, f);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  int left = nk_seg;  // k-tiles to the end of the segment
  auto segment = [&] {
    if constexpr (EPI == E_ACCUM) {
      if (--left == 0) {
        left = nk_seg;
        each([&](int i, int j, int r) {
          tot[i][j][r] += acc[i][j][r];
          acc[i][j][r] = 0.f;
        });
      }
    }
  };
  // requests the first three tiles and lays down the first
  auto begin = [&](auto stagec) {
    constexpr int CUR = decltype(stagec)::value;
    typedef std::integral_constant<int, CUR ^ 1> Next;
    aim(stagec);
#pragma unroll
    for (int c = 0; c < NC; ++c) load(stagec, c);
    aim(Next{});
#pragma unroll
    for (int c = 0; c < NC; ++c) load(Next{}, c);
    read_ahead();
#pragma unroll
    for (int c = 0; c < NC; ++c) store(stagec, CUR, c);
    aim(stagec);
#pragma unroll
    for (int c = 0; c < NC; ++c) load(stagec, c);
    __syncthreads();
#pragma unroll
    for (int f = 0; f < NF; ++f) fetch(0, CUR, 0, f);
  };
  static_assert(C::KW % 2 == 0, "an iteration ends with the fragment buffer it began with");
  begin(I0{});
  // Left in the middle after an odd number of tiles, and never joined there again: where paths with the loads of one set and
  // of both in flight meet, the compiler waits for both.
  for (int kt = nk;;) {
    iter(I0{});
    segment();
    if (--kt == 0) break;
    iter(I1{});
    segment();
    if (--kt == 0) break;
  }
  if constexpr (READS_R && !EARLY_R) read_r();
  each([&](int i, int j, int r) {
    if constexpr (EPI == E_ACCUM) {
      out.store(tot[i][j][r], i, j, r);
    } else if constexpr (EPI == E_BIAS_GELU) {
      const TO u = (TO)(acc[i][j][r] + bv[j]);
      out.store(u, i, j, r);
      out2.store((TO)gelu_f((float)u), i, j, r);
    } else {
      out.store((TO)epilogue_value<EPI>(acc[i][j][r], bv[j], READS_R ? rv[i][j][r] : 0.f), i, j, r);
    }
  });
}

// XCD x (workgroups go to the eight round-robin) gets a contiguous range of the tile order, so that the tiles that
// share its L2 share operand panels
__device__ __forceinline__ int tile_of_block() {
  const int lin = blockIdx.x;
  return (gridDim.x & 7) == 0 ? (lin & 7) * (int)(gridDim.x >> 3) + (lin >> 3) : lin;
}

template <typename C, typename TI, int VEC, bool AK, bool BKC, int EPI, typename TO>
__global__ __launch_bounds__(NT) void gemm_f32_kernel(int M, int N, int K, const TI* __restrict__ A, const TI* __restrict__ B,
                                                      TO* __restrict__ Cm, const float* __restrict__ bias, const TO* __restrict__ R,
                                                      TO* __restrict__ C2, int accumulate, int tiles_m, int n_seg, size_t seg_a,
                                                      size_t seg_b) {
  tile_product<C, TI, VEC, AK, BKC, EPI, TO>(tile_of_block(), M, N, K, A, B, Cm, bias, R, C2, accumulate, tiles_m, n_seg, seg_a, seg_b);
}

// The weight gradients of a stage in one launch.  In a small stack each has 64 to 256 tiles of a few microseconds, of which a
// launch, the first loads and the last stores are the most: one after the other they leave most of the chip idle.
struct Batch {
  struct Item {
    const float *A, *B;
    float* C;
    size_t seg_a, seg_b;
    int M, N, K, n_seg, accumulate, tiles_m, end;  // end: tiles of the items up to and with this one
  } it[GEMM_F32_BATCH];
};

template <typename C>
__global__ __launch_bounds__(NT) void gemm_f32_batch_kernel(Batch b) {
  const int lin = tile_of_block();
  int p = 0, first = 0;
  while (lin >= b.it[p].end) first = b.it[p++].end;
  const Batch::Item& t = b.it[p];
  tile_product<C, float, 4, false, false, E_ACCUM, float>(lin - first, t.M, t.N, t.K, t.A, t.B, t.C, nullptr, nullptr, nullptr, t.accumulate, t.tiles_m, t.n_seg,
                                                          t.seg_a, t.seg_b);
}

typedef Cfg<2, 2, 2, 2, 32, 32> CLarge;  // 128 x 128
typedef Cfg<2, 2, 2, 1, 32, 32> CTall;   // 128 x 64
typedef Cfg<2, 2, 1, 1, 32, 32> CMid;    // 64 x 64
typedef Cfg<2, 2, 1, 1, 64, 16> CSmall;  // 32 x 32

template <typename C, typename TI, int VEC, bool AK, bool BKC, int EPI, typename TO>
void launch(const GemmArgs& a, hipStream_t st) {
  const int tm = (a.M + C::BM - 1) / C::BM, tn = (a.N + C::BN - 1) / C::BN;
  gemm_f32_kernel<C, TI, VEC, AK, BKC, EPI, TO><<<(unsigned)tm * (unsigned)tn, NT, 0, st>>>(
      a.M, a.N, a.K, (const TI*)a.A, (const TI*)a.B, (TO*)a.C, a.bias, (const TO*)a.R, (TO*)a.C2, a.accumulate, tm, a.n_seg > 1 ? a.n_seg : 1,
      a.seg_stride_a, a.seg_stride_b);
}

// The matrix pipeline bounds every tile, so a product takes as long as the compute unit with the most tiles: tiles per
// unit (of 256) times the tile's area, plus what the smaller tiles lose between their k-tiles.
// n products of one launch share the rounds.
inline int choose(const GemmArgs* a, int n) {
  const int bm[4] = {128, 128, 64, 32}, bn[4] = {128, 64, 64, 32};
  const double rate[4] = {1.0, 0.95, 0.93, 0.78};
  int best = 0;
  double best_t = 0;
  for (int i = 0; i < 4; ++i) {
    long t = 0;
    for (int p = 0; p < n; ++p) t += (long)((a[p].M + bm[i] - 1) / bm[i]) * ((a[p].N + bn[i] - 1) / bn[i]);
    const double cost = (double)((t + 255) / 256) * bm[i] * bn[i] / rate[i];
    if (i == 0 || cost < best_t) { best = i; best_t = cost; }
  }
  return best;
}

template <typename TI, int VEC, bool AK, bool BKC, int EPI, typename TO>
void by_tile(const GemmArgs& a, hipStream_t st) {
  switch (choose(&a, 1)) {
    case 0: launch<CLarge, TI, VEC, AK, BKC, EPI, TO>(a, st); break;
    case 1: launch<CTall, TI, VEC, AK, BKC, EPI, TO>(a, st); break;
    case 2: launch<CMid, TI, VEC, AK, BKC, EPI, TO>(a, st); break;
    default: launch<CSmall, TI, VEC, AK, BKC, EPI, TO>(a, st); break;
  }
}

template <typename T, int VEC, bool AK, bool BKC>
bf_status by_epilogue(int epi, const GemmArgs& a, hipStream_t st) {
  if constexpr (!AK) {
    if (epi != E_ACCUM) { set_error("gemm: the weight-gradient layout stores fp32 with E_ACCUM only"); return BF_EINVAL; }
    by_tile<T, VEC, AK, BKC, E_ACCUM, float>(a, st);
  } else {
    switch (epi) {
      case E_NONE: by_tile<T, VEC, AK, BKC, E_NONE, T>(a, st); break;
      case E_BIAS: by_tile<T, VEC, AK, BKC, E_BIAS, T>(a, st); break;
      case E_BIAS_RES: by_tile<T, VEC, AK, BKC, E_BIAS_RES, T>(a, st); break;
      case E_BIAS_GELU: by_tile<T, VEC, AK, BKC, E_BIAS_GELU, T>(a, st); break;
      case E_GELU_BWD: by_tile<T, VEC, AK, BKC, E_GELU_BWD, T>(a, st); break;
      default: set_error("gemm: epilogue %d not available for this layout", epi); return BF_EINVAL;
    }
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_error("gemm_f32 launch failed: %s", hipGetErrorString(e)); return BF_EDEVICE; }
  return BF_OK;
}

template <typename T, int VEC>
bf_status by_layout(int layout, int epi, const GemmArgs& a, hipStream_t st) {
  if (layout == L_NN) return by_epilogue<T, VEC, true, false>(epi, a, st);
  if (layout == L_NT) return by_epilogue<T, VEC, true, true>(epi, a, st);
  return by_epilogue<T, VEC, false, false>(epi, a, st);
}

}  // namespace

bool gemm_f32_supported(int layout, int epi, const GemmArgs& a) {
  // 32-bit lane offsets: 128 rows of a K-contiguous operand, 64 k-rows of the other kind
  const long ldmax = 1l << 21;
  const long tiles = (long)((a.M + 31) / 32) * ((a.N + 31) / 32);
  return layout >= L_NN && layout <= L_TN && (layout == L_TN) == (epi == E_ACCUM) && a.M >= 1 && a.N >= 1 && a.K >= 1 && a.M <= ldmax &&
         a.N <= ldmax && (layout == L_TN || a.K <= ldmax) && tiles < (1l << 31) && (a.n_seg <= 1 || layout == L_TN);
}

// Where it is faster than the vector kernel (same bits): not a short contraction into a large output, which is bound by the
// epilogue, whose stores the vector kernel has four to a lane.  1416 x 16000, fp32, vector kernel / this: forward with
// residual K = 41 77 / 98 us, 72 94 / 104, 100 level; GeLU backward 69 / 104, 87 / 103, level; weight gradient 17 54 / 58, 65 92 / 88;
// bf16, plain epilogue 9 25 / 32, 17 34 / 31; up to 1000 x 1000 this one wins or is level throughout.
bool gemm_f32_better(int epi, const GemmArgs& a) {
  const int k_min = epi == E_NONE || epi == E_BIAS ? 17 : epi == E_ACCUM ? 48 : epi == E_BIAS_GELU ? 64 : epi == E_BIAS_RES ? 80 : 88;
  return a.K >= k_min || a.n_seg > 1 || (long)a.M * a.N < 2000000;
}

namespace {

template <typename C>
void launch_batch(const GemmArgs* a, int n, hipStream_t st) {
  Batch b{};
  int end = 0;
  for (int p = 0; p < n; ++p) {
    const int tm = (a[p].M + C::BM - 1) / C::BM, tn = (a[p].N + C::BN - 1) / C::BN;
    end += tm * tn;
    b.it[p] = {(const float*)a[p].A, (const float*)a[p].B, (float*)a[p].C, a[p].seg_stride_a, a[p].seg_stride_b,
               a[p].M, a[p].N, a[p].K, a[p].n_seg > 1 ? a[p].n_seg : 1, a[p].accumulate, tm, end};
  }
  gemm_f32_batch_kernel<C><<<(unsigned)end, NT, 0, st>>>(b);
}

// whole 16-byte chunks along the fast dimension of both operands
bool wide_chunks(int layout, const GemmArgs& a) {
  const int ra = layout == L_TN ? a.M : a.K, rb = layout == L_NT ? a.K : a.N;
  const size_t seg = a.n_seg > 1 ? a.seg_stride_a | a.seg_stride_b : 0;
  return ((ra | rb) & 3) == 0 && (seg & 3) == 0 && (((uintptr_t)a.A | (uintptr_t)a.B) & 15) == 0;
}

}  // namespace

// Every product of the batch would run here by itself, from wide chunks, and the tiles of all can be counted.
bool gemm_f32_batch_supported(const GemmArgs* a, int n) {
  long tiles = 0;
  for (int p = 0; p < n; ++p) {
    if (!gemm_f32_supported(L_TN, E_ACCUM, a[p]) || !gemm_f32_better(E_ACCUM, a[p]) || !wide_chunks(L_TN, a[p]) || a[p].colsum) return false;
    tiles += (long)((a[p].M + 31) / 32) * ((a[p].N + 31) / 32);
  }
  return n >= 1 && n <= GEMM_F32_BATCH && tiles < (1l << 31);
}

// The same bits as one launch each.  Stage of two fp32 layers of width 256 over 4 x 128 tokens: eight
// launches 54 us, one 24.
bf_status gemm_f32_batch(const GemmArgs* a, int n, hipStream_t st) {
  if (!gemm_f32_batch_supported(a, n)) { set_error("gemm_f32_batch: shapes not supported"); return BF_EINVAL; }
  for (int p = 0; p < n; ++p) {
    const bf_status s = gemm_check(L_TN, E_ACCUM, a[p]);
    if (s != BF_OK) return s;
  }
  switch (choose(a, n)) {
    case 0: launch_batch<CLarge>(a, n, st); break;
    case 1: launch_batch<CTall>(a, n, st); break;
    case 2: launch_batch<CMid>(a, n, st); break;
    default: launch_batch<CSmall>(a, n, st); break;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_error("gemm_f32_batch launch failed: %s", hipGetErrorString(e)); return BF_EDEVICE; }
  return BF_OK;
}

bf_status gemm_f32(int dtype, int layout, int epi, const GemmArgs& a, hipStream_t st) {
  if (!gemm_f32_supported(layout, epi, a)) { set_error("gemm_f32: shape not supported"); return BF_EINVAL; }
  if (dtype == BF_BF16) return by_layout<bf16_t, 1>(layout, epi, a, st);
  // element by element where there are no wide chunks
  return wide_chunks(layout, a) ? by_layout<float, 4>(layout, epi, a, st) : by_layout<float, 1>(layout, epi, a, st);
}

}  // namespace bf
