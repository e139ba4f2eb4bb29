// Fused attention on the gfx950 matrix cores: softmax(Q K^T / sqrt(S_head) [+ causal mask]) V
// forward, and its backward as two deterministic passes (dQ pass over key blocks, dK/dV pass
// over query blocks) that recompute the probabilities from the saved log-sum-exp.  No
// S_seq x S_seq tensor ever reaches HBM and nothing is accumulated with atomics, so the
// result does not depend on scheduling.
//
// Every score tile is computed TRANSPOSED where that keeps "one lane = one softmax row":
//   forward / dQ pass:  S^T = K Q^T   (MFMA rows = keys,    columns = the wave's 32 queries)
//   dK/dV pass:         S   = Q K^T   (MFMA rows = queries, columns = the wave's 32 keys)
// In the accumulator layout of v_mfma_f32_32x32x16_bf16 (lane l, register r holds
// row (r/4)*8 + (l/32)*4 + r%4, column l%32) a lane then owns one column and 16 rows, so a
// row statistic of the softmax is a per-lane scalar (forward) and the 8 registers
// 8kk..8kk+7 of a lane, rounded to bf16, are directly the B operand of the next product
// for the contraction rows 16kk + 8(e/4) + 4(l/32) + e%4.  The matching A operand is read
// from LDS with the transpose load (ds_read_b64_tr_b16) using that same row order.
//
// LDS tiles are [row][S_head] with the 16-byte chunk index XOR-swizzled by row bits; the
// layout serves both the K-contiguous 16-byte fragment reads and the transpose loads without
// bank conflicts.
#include <float.h>

#include <algorithm>
#include <type_traits>

#include "attention_tiles.h"
#include "common.h"

namespace bf {

namespace {

// Register set that carries tile j+1, from the parity of j: a compile-time constant when the loop
// is unrolled by two (the parity is an integral_constant), always set 0 with one tile in flight.
template <int DEPTH, typename P>
struct NextSetOf { static constexpr int value = 0; };
template <int DEPTH, int V>
struct NextSetOf<DEPTH, std::integral_constant<int, V>> { static constexpr int value = (V + 1) % DEPTH; };

// ------------------------------------------------------------------------------ forward
// ROWS queries per workgroup (one wave per 32): 128 with 4 waves and two workgroups per compute
// unit, or 256 with 8 waves and one.  The K/V tiles come through registers DEPTH tiles ahead of
// their use and are double-buffered in LDS: tile j+1 is written to the idle stage while tile j is
// consumed, so an iteration has a single barrier.  The 256-query form reads each tile from HBM / L2
// once for twice as many queries and keeps two tiles in flight; it needs enough (head, block) pairs
// to fill the chip.
// Measured at S_seq 1024-2048, 64 heads of 128: timed without softmax, P V and K/V refetch, the bare
// S = K Q^T loop (one 1 KB LDS fragment read per MFMA, Q from registers) reaches 44 % of the MFMA
// rate; without P V 70 % of the full time remains, without the softmax arithmetic 84 %, without the
// K/V refetch 86 %: no single part dominates, the per-tile chain read -> MFMA -> softmax -> MFMA is
// what two wavefronts per SIMD cannot hide.  Fewer LDS bytes per MFMA need 64 queries per wavefront
// (accumulators in AGPRs, one wavefront per SIMD): built and measured level with this form (100 against
// 98 us at 64 heads of 128, S_seq 2048): a lone wavefront issues in order, so each of its LDS, barrier
// and softmax waits stops its MFMAs too, and there is no partner on the SIMD to fill the gap.
template <int D, int ROWS>
__global__ __launch_bounds__(2 * ROWS, ROWS == 128 ? 2 : 1) void attn_fwd_kernel(const bf16_t* __restrict__ qkv,
                                                                                 bf16_t* __restrict__ ctx, float* __restrict__ lse,
                                                                                 int S_seq, int N_heads, int S_mb, int causal,
                                                                                 float scale) {
  constexpr int NT = 2 * ROWS, DEPTH = ROWS == 128 ? 1 : 2;
  __shared__ __attribute__((aligned(16))) bf16_t KVs[2][2][BLK * D];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  // 1-D grid ordered by work: the last (longest) query block of every head first, then the next ...
  const int nhb = N_heads * S_mb;
  const int qblk = S_seq / ROWS - 1 - blockIdx.x / nhb;
  const int head = (blockIdx.x % nhb) % N_heads, b = (blockIdx.x % nhb) / N_heads;
  const int h = N_heads * D;
  const size_t ld = 3 * (size_t)h;
  const bf16_t* base = qkv + (size_t)b * S_seq * ld + head * D;
  const int q0 = qblk * ROWS, qw = q0 + 32 * w, q = qw + (lane & 31);

  FragAddr<D> fa;
  fa.init(lane);
  bf16x8 qf[D / 16];
  load_rowfrags<D>(base + (size_t)q * ld, lane, qf);
  f32x16 o[D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt) o[dt] = zero16();
  // The running maximum starts at the lowest finite value: while a row has met only scores of -inf, from
  // -inf or overflowing keys, their difference to it is -inf and adds exactly 0, where -inf - -inf would be a NaN.
  float m = -FLT_MAX, l = 0.f;
  const float c2 = scale * LOG2E;

  const int nblk = causal ? (q0 + ROWS) / BLK : S_seq / BLK;
  TileRegs<BLK, D, NT> kr[DEPTH], vr[DEPTH];  // set (j % DEPTH) carries tile j
  auto fetch = [&](auto setc, int j) {
    constexpr int SET = decltype(setc)::value;
    kr[SET].load(base + (size_t)j * BLK * ld + h, ld, tid);
    vr[SET].load(base + (size_t)j * BLK * ld + 2 * h, ld, tid);
  };
  typedef std::integral_constant<int, 0> I0;
  typedef std::integral_constant<int, 1> I1;
  fetch(I0{}, 0);
  kr[0].store(KVs[0][0], tid);
  vr[0].store(KVs[0][1], tid);
  if (nblk > 1) fetch(std::integral_constant<int, 1 % DEPTH>{}, 1);
  if (DEPTH > 1 && nblk > 2) fetch(I0{}, 2);
  __syncthreads();
  // one key tile; PAR = j & 1 is a compile-time constant (the loop is unrolled by two) so that the
  // LDS stage and the register set are too
  auto body = [&](int j, auto parc) {
    constexpr int PAR = decltype(parc)::value;
    typedef std::integral_constant<int, (PAR + 1) % DEPTH> NextSet;
    const bf16_t* Ks = KVs[PAR][0];
    const bf16_t* Vs = KVs[PAR][1];
    if (j + 1 < nblk) {
      kr[NextSet::value].store(KVs[PAR ^ 1][0], tid);
      vr[NextSet::value].store(KVs[PAR ^ 1][1], tid);
    }
    if (j + 1 + DEPTH < nblk) fetch(NextSet{}, j + 1 + DEPTH);
    const int kb = j * BLK;
    if (causal && kb > qw + 31) { __syncthreads(); return; }  // the whole tile is above this wave's diagonal
    f32x16 s[2] = {zero16(), zero16()};
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk)
#pragma unroll
      for (int t = 0; t < 2; ++t)
        s[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa.frag_k(Ks, 32 * t, kk), qf[kk], s[t], 0, 0, 0);
    mfma_lds_pipeline<2 * (D / 16), 1, 4>();
    // Online softmax on the raw scores: m is the running max of the unscaled scores, the scale
    // 1/sqrt(S_head) log2(e) enters through one fma per element, the exponentials are the
    // hardware exp2 (arguments <= 0; masked scores are -inf and give exactly 0).
    if (causal && kb + BLK - 1 > qw) {  // only tiles that touch the diagonal pay for the mask
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (kb + 32 * t + acc_row(r, lane) > q) s[t][r] = -INFINITY;
    }
    float mx = m;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[t][r]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float nmx = -mx * c2;
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = __builtin_amdgcn_exp2f(fmaf(s[t][r], c2, nmx));
        s[t][r] = p;
        sum += p;
      }
    if (__builtin_amdgcn_ballot_w64(mx > m) != 0) {  // some row's max moved: rescale (rare after the first tiles)
      const float alpha = __builtin_amdgcn_exp2f(fmaf(m, c2, nmx));
      l *= alpha;
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
      m = mx;
    }
    l += sum;
    bf16x8 pb[2][2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int k2 = 0; k2 < 2; ++k2) pb[t][k2] = pack8(s[t], k2);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt)
          o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa.frag_t(Vs, 32 * t + 16 * k2, dt), pb[t][k2], o[dt], 0, 0, 0);
    mfma_lds_pipeline<4 * (D / 32), 2, 4>();
    __syncthreads();
  };
  for (int j = 0; j < nblk; j += 2) {
    body(j, I0{});
    if (j + 1 < nblk) body(j + 1, I1{});
  }
  l += __shfl_xor(l, 32, 64);
  store_rows<D>(o, ctx + ((size_t)b * S_seq + q) * h + head * D, lane, 1.0f / l);
  if (lane < 32) lse[((size_t)b * N_heads + head) * S_seq + q] = m * scale + logf(l);
}

// The forward kernel's other forms: any length (EDGE: the last tile and the last rows partly empty), and two groups of waves
// that take every other key tile of the same rows (KG = 2, tiles staged in pairs) and merge their maxima, sums and outputs
// in LDS at the end, for launches of few rows.  A kernel of its own: as parameters of the one above the two changed the
// schedule of its common form (S_head 64, S_seq 512, 100 heads, causal 13.0 -> 14.5 us; 128, 1152, 64 heads, bidirectional
// 70.8 -> 75.2), which is why their bodies, alike as they are, stay apart.
template <int D, int ROWS, bool EDGE, int KG>
__global__ __launch_bounds__(2 * ROWS * KG, ROWS == 128 && !(EDGE && D == 128 && KG == 1) ? 2 : 1) void attn_fwd_general_kernel(const bf16_t* __restrict__ qkv,
                                                                                 bf16_t* __restrict__ ctx, float* __restrict__ lse,
                                                                                 int S_seq, int N_heads, int S_mb, int causal,
                                                                                 float scale) {
  static_assert((EDGE || KG == 2) && ROWS <= 128, "whole lengths with one key group have a kernel of their own");
  constexpr int NT = 2 * ROWS * KG, BT = BLK * KG;
  __shared__ __attribute__((aligned(16))) bf16_t KVs[2][2][BT * D];
  const int tid = threadIdx.x, lane = tid & 63;
  const int grp = KG == 1 ? 0 : (tid >> 6) / (ROWS / 32), w = KG == 1 ? tid >> 6 : (tid >> 6) % (ROWS / 32);  // key group, rows
  // 1-D grid ordered by work: the last (longest) query block of every head first, then the next ...
  const int nhb = N_heads * S_mb;
  const int qblk = (EDGE ? (S_seq + ROWS - 1) / ROWS : S_seq / ROWS) - 1 - blockIdx.x / nhb;
  const int head = (blockIdx.x % nhb) % N_heads, b = (blockIdx.x % nhb) / N_heads;
  const int h = N_heads * D;
  const size_t ld = 3 * (size_t)h;
  const bf16_t* base = qkv + (size_t)b * S_seq * ld + head * D;
  const int q0 = qblk * ROWS, qw = q0 + 32 * w, q = qw + (lane & 31);
  const int ql = EDGE ? min(q, S_seq - 1) : q;  // the row that is read in the place of q
  __shared__ float dump[EDGE ? NT / 64 * DUMP : 1];
  __shared__ int bad_tile[2];  // per LDS stage: 1 + the last tile staged there with a non-finite V
  if (EDGE && tid < 2) bad_tile[tid] = 0;

  FragAddr<D> fa;
  fa.init(lane);
  bf16x8 qf[D / 16];
  load_rowfrags<D>(base + (size_t)ql * ld, lane, qf);
  f32x16 o[D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt) o[dt] = zero16();
  // The running maximum starts at the lowest finite value: while a row (or a key group's share of it) has met only scores of -inf, from
  // -inf or overflowing keys, their difference to it is -inf and adds exactly 0, where -inf - -inf would be a NaN.
  float m = -FLT_MAX, l = 0.f;
  // EDGE: the exponent is the difference to the maximum times its factor, so that no rounding of the maximum enters every
  // term and the log-sum-exp; where 1/sqrt(S_head) is no power of two the scores are scaled first, as the fp32 kernels do
  // it, and no rounding of scale x log2(e) does either (log-sum-exp over 1000 keys: off by 4.8e-8 -> 4.3e-8, those kernels 4.4e-8)
  constexpr bool SCALED = EDGE && D == 128;
  const float c2 = SCALED ? LOG2E : scale * LOG2E;

  const int nblk = EDGE ? ((causal ? min(q0 + ROWS, S_seq) : S_seq) + BT - 1) / BT : causal ? (q0 + ROWS + (KG - 1) * BLK) / BT : S_seq / BT;
  TileRegs<BT, D, NT> kr, vr;
  auto fetch = [&](int j) {
    if constexpr (EDGE) {
      kr.load_edge(base + (size_t)j * BT * ld + h, ld, tid, S_seq - j * BT);
      vr.load_edge(base + (size_t)j * BT * ld + 2 * h, ld, tid, S_seq - j * BT);
      return;
    }
    kr.load(base + (size_t)j * BT * ld + h, ld, tid);
    vr.load(base + (size_t)j * BT * ld + 2 * h, ld, tid);
  };
  typedef std::integral_constant<int, 0> I0;
  typedef std::integral_constant<int, 1> I1;
  fetch(0);
  // tile j goes to an LDS stage: does it hold what must not meet a masked zero or a probability's smaller parts
  auto note = [&](int j, int stage, const TileRegs<BT, D, NT>& v) {
    if (EDGE && v.non_finite()) bad_tile[stage] = j + 1;
  };
  if (EDGE) __syncthreads();  // bad_tile is clear
  kr.store(KVs[0][0], tid);
  vr.store(KVs[0][1], tid);
  note(0, 0, vr);
  if (nblk > 1) fetch(1);
  __syncthreads();
  // one key tile; PAR = j & 1, the LDS stage, is a compile-time constant (the loop is unrolled by two)
  auto body = [&](int j, auto parc) {
    constexpr int PAR = decltype(parc)::value;
    const bf16_t* Ks = KVs[PAR][0] + grp * BLK * D;
    const bf16_t* Vs = KVs[PAR][1] + grp * BLK * D;
    if (j + 1 < nblk) {
      kr.store(KVs[PAR ^ 1][0], tid);
      vr.store(KVs[PAR ^ 1][1], tid);
      note(j + 1, PAR ^ 1, vr);
    }
    if (j + 2 < nblk) fetch(j + 2);
    const int kb = j * BT + grp * BLK;
    // the whole tile is above this wave's diagonal, or the wave's rows are past the end
    if ((causal && kb > qw + 31) || (EDGE && (qw >= S_seq || kb >= S_seq))) { __syncthreads(); return; }
    f32x16 s[2] = {zero16(), zero16()};
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk)
#pragma unroll
      for (int t = 0; t < 2; ++t)
        s[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa.frag_k(Ks, 32 * t, kk), qf[kk], s[t], 0, 0, 0);
    mfma_lds_pipeline<2 * (D / 16), 1, 4>();
    // Online softmax on the raw scores: m is the running max of the unscaled scores, the scale
    // 1/sqrt(S_head) log2(e) enters through one fma per element, the exponentials are the
    // hardware exp2 (arguments <= 0; masked scores are -inf and give exactly 0).
    if (causal && kb + BLK - 1 > qw) {  // only tiles that touch the diagonal pay for the mask
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (kb + 32 * t + acc_row(r, lane) > q) s[t][r] = -INFINITY;
    }
    if (EDGE && kb + BLK > S_seq) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (kb + 32 * t + acc_row(r, lane) >= S_seq) s[t][r] = -INFINITY;
    }
    if (SCALED) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[t][r] *= scale;
    }
    float mx = m;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[t][r]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float nmx = -mx * c2;
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = __builtin_amdgcn_exp2f(EDGE ? (s[t][r] - mx) * c2 : fmaf(s[t][r], c2, nmx));
        s[t][r] = p;
        sum += p;
      }
    if (__builtin_amdgcn_ballot_w64(mx > m) != 0) {  // some row's max moved: rescale (rare after the first tiles)
      const float alpha = __builtin_amdgcn_exp2f(EDGE ? (m - mx) * c2 : fmaf(m, c2, nmx));
      l *= alpha;
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
      m = mx;
    }
    l += sum;
    if constexpr (EDGE) {
      if (bad_tile[PAR] == j + 1) {
        accumulate_allowed<D, 2>(o, s, 0, Vs, dump + (tid >> 6) * DUMP, lane, [&](int row) { return (!causal || kb + row <= q) && kb + row < S_seq; });
        __syncthreads();
        return;
      }
#pragma unroll
      for (int t = 0; t < 2; ++t) accumulate_split<D>(o, s[t], Vs, 32 * t, fa);
      __syncthreads();
      return;
    }
    bf16x8 pb[2][2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int k2 = 0; k2 < 2; ++k2) pb[t][k2] = pack8(s[t], k2);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt)
          o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa.frag_t(Vs, 32 * t + 16 * k2, dt), pb[t][k2], o[dt], 0, 0, 0);
    mfma_lds_pipeline<4 * (D / 32), 2, 4>();
    __syncthreads();
  };
  for (int j = 0; j < nblk; j += 2) {
    body(j, I0{});
    if (j + 1 < nblk) body(j + 1, I1{});
  }
  if constexpr (KG == 2) {
    // the second key group hands its rows over, lane to lane (the loop ended on a barrier: the tiles are free); it may
    // have seen no finite score (maximum -FLT_MAX, sums 0)
    constexpr int NV = D / 2 + 2;
    static_assert(NV * 64 * (ROWS / 32) * 4 <= sizeof(KVs), "the hand-over does not fit");
    float* hb = reinterpret_cast<float*>(&KVs[0][0][0]) + w * NV * 64 + lane;
    if (grp == 1) {
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) hb[(dt * 16 + r) * 64] = o[dt][r];
      hb[(NV - 2) * 64] = m;
      hb[(NV - 1) * 64] = l;
    }
    __syncthreads();
    if (grp == 1) return;
    const float m1 = hb[(NV - 2) * 64], M = fmaxf(m, m1);
    const float a0 = __builtin_amdgcn_exp2f((m - M) * c2), a1 = __builtin_amdgcn_exp2f((m1 - M) * c2);
    l = l * a0 + hb[(NV - 1) * 64] * a1;
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[dt][r] = o[dt][r] * a0 + hb[(dt * 16 + r) * 64] * a1;
    m = M;
  }
  l += __shfl_xor(l, 32, 64);
  if (EDGE && q >= S_seq) return;
  store_rows<D>(o, ctx + ((size_t)b * S_seq + q) * h + head * D, lane, 1.0f / l);
  if (lane < 32) lse[((size_t)b * N_heads + head) * S_seq + q] = (SCALED ? m : m * scale) + logf(l);
}

// ------------------------------------------------------------------- backward, dQ pass
// Also takes delta[b, head, i] = sum_c dctx[i, c] ctx[i, c] of its queries (each lane already holds
// half of its query's dctx row) and leaves it in `delta` for the dK/dV pass.
// ROWS queries per workgroup and K/V tiles DEPTH tiles ahead, as in the forward kernel.
template <int D, int ROWS>
__global__ __launch_bounds__(2 * ROWS, ROWS == 128 ? 2 : 1) void attn_bwd_dq_kernel(
    const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ ctx, const bf16_t* __restrict__ dctx,
    const float* __restrict__ lse, float* __restrict__ delta, bf16_t* __restrict__ dqkv, int S_seq, int N_heads, int S_mb,
    int causal, float scale, float* __restrict__ colpart) {
  constexpr int NT = 2 * ROWS, DEPTH = ROWS == 128 ? 1 : 2;
  __shared__ __attribute__((aligned(16))) bf16_t KVs[2][2][BLK * D];  // double-buffered, one barrier per tile
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int nhb = N_heads * S_mb;
  const int qblk = S_seq / ROWS - 1 - blockIdx.x / nhb;  // longest query blocks of every head first
  const int head = (blockIdx.x % nhb) % N_heads, b = (blockIdx.x % nhb) / N_heads;
  const int h = N_heads * D;
  const size_t ld = 3 * (size_t)h;
  const bf16_t* base = qkv + (size_t)b * S_seq * ld + head * D;
  const int q0 = qblk * ROWS, qw = q0 + 32 * w, q = qw + (lane & 31);

  // precomputed offsets where the registers allow (the 128-query form at S_head 128 would spill)
  typename std::conditional<(ROWS == 256 || D == 64), FragAddr<D>, FragAddrLive<D>>::type fa;
  fa.init(lane);
  bf16x8 qf[D / 16], dof[D / 16];
  load_rowfrags<D>(base + (size_t)q * ld, lane, qf);
  load_rowfrags<D>(dctx + ((size_t)b * S_seq + q) * h + head * D, lane, dof);
  const size_t st = ((size_t)b * N_heads + head) * S_seq + q;
  float dl = 0.f;
  {
    bf16x8 cf[D / 16];
    load_rowfrags<D>(ctx + ((size_t)b * S_seq + q) * h + head * D, lane, cf);
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk)
#pragma unroll
      for (int e = 0; e < 8; ++e) dl = fmaf((float)dof[kk][e], (float)cf[kk][e], dl);
    dl += __shfl_xor(dl, 32, 64);  // lanes l and l + 32 hold the two halves of the row
    if (lane < 32) delta[st] = dl;
  }
  const float lse2 = lse[st] * LOG2E, c2 = scale * LOG2E;
  f32x16 dq[D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt) dq[dt] = zero16();

  const int nblk = causal ? (q0 + ROWS) / BLK : S_seq / BLK;
  TileRegs<BLK, D, NT> kr[DEPTH], vr[DEPTH];  // set (j % DEPTH) carries tile j
  auto fetch = [&](auto setc, int j) {
    constexpr int SET = decltype(setc)::value;
    kr[SET].load(base + (size_t)j * BLK * ld + h, ld, tid);
    vr[SET].load(base + (size_t)j * BLK * ld + 2 * h, ld, tid);
  };
  typedef std::integral_constant<int, 0> I0;
  typedef std::integral_constant<int, 1> I1;
  fetch(I0{}, 0);
  kr[0].store(KVs[0][0], tid);
  vr[0].store(KVs[0][1], tid);
  if (nblk > 1) fetch(std::integral_constant<int, 1 % DEPTH>{}, 1);
  if (DEPTH > 1 && nblk > 2) fetch(I0{}, 2);
  __syncthreads();
  // one key tile; par = j & 1 selects the LDS stage
  auto body = [&](int j, auto par) {
    typedef std::integral_constant<int, NextSetOf<DEPTH, decltype(par)>::value> NextSet;
    const int p = par;
    const bf16_t* Ks = KVs[p][0];
    const bf16_t* Vs = KVs[p][1];
    if (j + 1 < nblk) {
      kr[NextSet::value].store(KVs[p ^ 1][0], tid);
      vr[NextSet::value].store(KVs[p ^ 1][1], tid);
    }
    if (j + 1 + DEPTH < nblk) fetch(NextSet{}, j + 1 + DEPTH);
    const int kb = j * BLK;
    if (causal && kb > qw + 31) { __syncthreads(); return; }
    const bool diag = causal && kb + BLK - 1 > qw;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      f32x16 s = zero16(), dp = zero16();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kk = 0; kk < D / 16; ++kk) {
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa.frag_k(Ks, 32 * t, kk), qf[kk], s, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa.frag_k(Vs, 32 * t, kk), dof[kk], dp, 0, 0, 0);
      }
      mfma_lds_pipeline<2 * (D / 16), 1, 4>();
      // p = exp(s/sqrt(d) - lse); dS = p (dP - delta) (the factor 1/sqrt(d) is applied once, to dQ)
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c2, -lse2)) * (dp[r] - dl);
      if (diag) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (kb + 32 * t + acc_row(r, lane) > q) s[r] = 0.f;
      }
      const bf16x8 dsb[2] = {pack8(s, 0), pack8(s, 1)};
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt)
          dq[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa.frag_t(Ks, 32 * t + 16 * k2, dt), dsb[k2], dq[dt], 0, 0, 0);
      mfma_lds_pipeline<2 * (D / 32), 2, 4>();
    }
    __syncthreads();
  };
  if constexpr (ROWS == 256 || D == 64) {
    // unrolled by two: the LDS stage (and with it every fragment address) is a compile-time constant
    for (int j = 0; j < nblk; j += 2) {
      body(j, I0{});
      if (j + 1 < nblk) body(j + 1, I1{});
    }
  } else {
    static_assert(DEPTH == 1, "a run-time stage goes with one tile in flight");
    for (int j = 0; j < nblk; ++j) body(j, j & 1);
  }
  store_rows<D>(dq, dqkv + ((size_t)b * S_seq + q) * ld + head * D, lane, scale);
  if (colpart) {
    // row (b, query block) of the partial column sums of dQ, [S_mb * S_seq / ROWS][N_heads * D]; the tile
    // buffers are free: the loop ended on a barrier
    float* red = reinterpret_cast<float*>(&KVs[0][0][0]);
    wave_colsum<D>(dq, scale, red + (size_t)w * 4 * (D / 2), lane);
    __syncthreads();
    if (tid < D) colpart[((size_t)b * (S_seq / ROWS) + qblk) * h + head * D + tid] = colsum_of<D>(red, 0, NT / 64, tid);
  }
}

// The dQ kernel's other forms, as in the forward pass.
template <int D, int ROWS, bool EDGE, int KG>
__global__ __launch_bounds__(2 * ROWS * KG, ROWS == 128 && !EDGE ? 2 : 1) void attn_bwd_dq_general_kernel(
    const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ ctx, const bf16_t* __restrict__ dctx,
    const float* __restrict__ lse, float* __restrict__ delta, bf16_t* __restrict__ dqkv, int S_seq, int N_heads, int S_mb,
    int causal, float scale, float* __restrict__ colpart) {
  static_assert((EDGE || KG == 2) && ROWS <= 128, "whole lengths with one key group have a kernel of their own");
  constexpr int NT = 2 * ROWS * KG, BT = BLK * KG;
  __shared__ __attribute__((aligned(16))) bf16_t KVs[2][2][BT * D];  // double-buffered, one barrier per tile
  const int tid = threadIdx.x, lane = tid & 63;
  const int grp = KG == 1 ? 0 : (tid >> 6) / (ROWS / 32), w = KG == 1 ? tid >> 6 : (tid >> 6) % (ROWS / 32);  // key group, rows
  const int nhb = N_heads * S_mb;
  const int qblk = (EDGE ? (S_seq + ROWS - 1) / ROWS : S_seq / ROWS) - 1 - blockIdx.x / nhb;  // longest query blocks of every head first
  const int head = (blockIdx.x % nhb) % N_heads, b = (blockIdx.x % nhb) / N_heads;
  const int h = N_heads * D;
  const size_t ld = 3 * (size_t)h;
  const bf16_t* base = qkv + (size_t)b * S_seq * ld + head * D;
  const int q0 = qblk * ROWS, qw = q0 + 32 * w, q = qw + (lane & 31);
  const int ql = EDGE ? min(q, S_seq - 1) : q;  // the row that is read in the place of q
  __shared__ float dump[EDGE ? NT / 64 * DUMP : 1];
  __shared__ int bad_tile[2];  // per LDS stage: 1 + the last tile staged there with a non-finite K
  if (EDGE && tid < 2) bad_tile[tid] = 0;

  FragAddr<D> fa;
  fa.init(lane);
  bf16x8 qf[D / 16], dof[D / 16];
  load_rowfrags<D>(base + (size_t)ql * ld, lane, qf);
  load_rowfrags<D>(dctx + ((size_t)b * S_seq + ql) * h + head * D, lane, dof);
  const size_t st = ((size_t)b * N_heads + head) * S_seq + ql;
  float dl = 0.f;
  {
    bf16x8 cf[D / 16];
    load_rowfrags<D>(ctx + ((size_t)b * S_seq + ql) * h + head * D, lane, cf);
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk)
#pragma unroll
      for (int e = 0; e < 8; ++e) dl = fmaf((float)dof[kk][e], (float)cf[kk][e], dl);
    dl += __shfl_xor(dl, 32, 64);  // lanes l and l + 32 hold the two halves of the row
    if (lane < 32 && grp == 0 && (!EDGE || q < S_seq)) delta[st] = dl;
  }
  const float lse2 = lse[st] * LOG2E, c2 = scale * LOG2E;
  f32x16 dq[D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt) dq[dt] = zero16();

  const int nblk = EDGE ? ((causal ? min(q0 + ROWS, S_seq) : S_seq) + BT - 1) / BT : causal ? (q0 + ROWS + (KG - 1) * BLK) / BT : S_seq / BT;
  TileRegs<BT, D, NT> kr, vr;
  auto fetch = [&](int j) {
    if constexpr (EDGE) {
      kr.load_edge(base + (size_t)j * BT * ld + h, ld, tid, S_seq - j * BT);
      vr.load_edge(base + (size_t)j * BT * ld + 2 * h, ld, tid, S_seq - j * BT);
      return;
    }
    kr.load(base + (size_t)j * BT * ld + h, ld, tid);
    vr.load(base + (size_t)j * BT * ld + 2 * h, ld, tid);
  };
  typedef std::integral_constant<int, 0> I0;
  typedef std::integral_constant<int, 1> I1;
  fetch(0);
  auto note = [&](int j, int stage, const TileRegs<BT, D, NT>& k) {
    if (EDGE && k.non_finite()) bad_tile[stage] = j + 1;
  };
  if (EDGE) __syncthreads();  // bad_tile is clear
  kr.store(KVs[0][0], tid);
  vr.store(KVs[0][1], tid);
  note(0, 0, kr);
  if (nblk > 1) fetch(1);
  __syncthreads();
  // one key tile; p = j & 1, the LDS stage, is a compile-time constant (the loop is unrolled by two)
  auto body = [&](int j, auto parc) {
    constexpr int p = decltype(parc)::value;
    const bf16_t* Ks = KVs[p][0] + grp * BLK * D;
    const bf16_t* Vs = KVs[p][1] + grp * BLK * D;
    if (j + 1 < nblk) {
      kr.store(KVs[p ^ 1][0], tid);
      vr.store(KVs[p ^ 1][1], tid);
      note(j + 1, p ^ 1, kr);
    }
    if (j + 2 < nblk) fetch(j + 2);
    const int kb = j * BT + grp * BLK;
    if ((causal && kb > qw + 31) || (EDGE && (qw >= S_seq || kb >= S_seq))) { __syncthreads(); return; }
    const bool diag = causal && kb + BLK - 1 > qw;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      f32x16 s = zero16(), dp = zero16();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kk = 0; kk < D / 16; ++kk) {
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa.frag_k(Ks, 32 * t, kk), qf[kk], s, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa.frag_k(Vs, 32 * t, kk), dof[kk], dp, 0, 0, 0);
      }
      mfma_lds_pipeline<2 * (D / 16), 1, 4>();
      // p = exp(s/sqrt(d) - lse); dS = p (dP - delta) (the factor 1/sqrt(d) is applied once, to dQ)
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c2, -lse2)) * (dp[r] - dl);
      if (diag) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (kb + 32 * t + acc_row(r, lane) > q) s[r] = 0.f;
      }
      if constexpr (EDGE) {
        if (kb + BLK > S_seq) {
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (kb + 32 * t + acc_row(r, lane) >= S_seq) s[r] = 0.f;
        }
        const f32x16 s1[1] = {s};
        if (bad_tile[p] == j + 1 || past_bf16(s1)) {
          accumulate_allowed<D, 1>(dq, s1, t, Ks, dump + (tid >> 6) * DUMP, lane, [&](int row) { return (!causal || kb + row <= q) && kb + row < S_seq; });
          continue;
        }
        accumulate_split<D>(dq, s, Ks, 32 * t, fa);
        continue;
      }
      const bf16x8 dsb[2] = {pack8(s, 0), pack8(s, 1)};
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt)
          dq[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa.frag_t(Ks, 32 * t + 16 * k2, dt), dsb[k2], dq[dt], 0, 0, 0);
      mfma_lds_pipeline<2 * (D / 32), 2, 4>();
    }
    __syncthreads();
  };
  for (int j = 0; j < nblk; j += 2) {
    body(j, I0{});
    if (j + 1 < nblk) body(j + 1, I1{});
  }
  if constexpr (KG == 2) {
    // the second key group's share, lane to lane
    constexpr int NV = D / 2;
    static_assert(NV * 64 * (ROWS / 32) * 4 <= sizeof(KVs), "the hand-over does not fit");
    float* hb = reinterpret_cast<float*>(&KVs[0][0][0]) + w * NV * 64 + lane;
    if (grp == 1) {
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) hb[(dt * 16 + r) * 64] = dq[dt][r];
    }
    __syncthreads();
    if (grp == 0) {
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) dq[dt][r] += hb[(dt * 16 + r) * 64];
    }
    __syncthreads();  // the hand-over has been read: the column sums below use the same LDS
  }
  if (EDGE && q >= S_seq) return;
  if (grp == 0) store_rows<D>(dq, dqkv + ((size_t)b * S_seq + q) * ld + head * D, lane, scale);
  if (colpart) {
    // row (b, query block) of the partial column sums of dQ, [S_mb * S_seq / ROWS][N_heads * D]; the tile
    // buffers are free: the loop ended on a barrier
    float* red = reinterpret_cast<float*>(&KVs[0][0][0]);
    if (grp == 0) wave_colsum<D>(dq, scale, red + (size_t)w * 4 * (D / 2), lane);
    __syncthreads();
    if (tid < D) colpart[((size_t)b * (S_seq / ROWS) + qblk) * h + head * D + tid] = colsum_of<D>(red, 0, ROWS / 32, tid);
  }
}

// ----------------------------------------------------------------- backward, dK/dV pass
// 8 waves per 128-key block, in pairs: waves 0-3 (one per 32 keys) accumulate dV = P^T dO, waves 4-7 the
// matching dK = dS^T Q.  The pair shares the probabilities: the dV wave computes S = Q K^T and
// P = exp(S / sqrt(d) - lse), keeps P (rounded to bf16, as its MFMA operand) and hands it to its
// partner through LDS, lane to lane (both hold the same 32 x 32 accumulator layout); the dK wave
// computes dP = dO V^T meanwhile and forms dS = P (dP - delta).  Each role runs two score-sized
// products per sub-tile and holds one 32 x S_head accumulator set plus its own K or V rows in
// registers, which leaves room for precomputed fragment addresses: two waves share a SIMD and one
// role's exponentials overlap the other's MFMAs.
// EDGE: the three parts of a probability take those registers (S_head 128: 12 scratch reads per sub-tile with them, 3 with
// addresses from two registers).  QG = 2: 64 keys a workgroup, waves 2, 3, 6 and 7 take the second half of every query tile and
// their sums are added at the end; bound by the same chain, but the longest key block is half as long.  2 x 1000 tokens, 16 heads of
// 128, causal, this pass: 112 us, about 100 without branches around the score gradients and with the addresses from two registers, 68 with QG = 2.
constexpr int NTHR_DKV = 512;

// S_head 64: two workgroups per compute unit want at most 128 registers, one fewer than the compiler takes by itself
// (4 x 1024 tokens, 16 heads, bidirectional: 70 -> 53 us).
template <int D, bool EDGE = false, int QG = 1>
__global__ __launch_bounds__(NTHR_DKV, D == 64 && !EDGE ? 4 : 2) void attn_bwd_dkv_kernel(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ dctx,
                                                                const float* __restrict__ lse, const float* __restrict__ delta,
                                                                bf16_t* __restrict__ dqkv, int S_seq, int N_heads, int S_mb, int causal,
                                                                float scale, float* __restrict__ colpart) {
  static_assert(QG == 1 || (QG == 2 && EDGE), "whole lengths have one query group");
  constexpr int KEYS = WG_ROWS / QG, KGS = KEYS / 32;  // keys of the workgroup, and groups of 32 of them
  __shared__ __attribute__((aligned(16))) bf16_t QOs[2][2][BLK * D];  // Q and dO tiles, double-buffered
  __shared__ __attribute__((aligned(16))) float stat_s[2][2][BLK];    // lse * log2(e) and delta of the tile's queries
  // P of a sub-tile, in bf16 [sub-tile][key group][register half][lane]; EDGE: in fp32 [sub-tile][key group][register quarter][lane]
  __shared__ __attribute__((aligned(16))) bf16_t Ps[EDGE ? 1 : 2][EDGE ? 1 : 4][EDGE ? 1 : 2][EDGE ? 8 : 64 * 8];
  __shared__ __attribute__((aligned(16))) float Pf[EDGE ? 2 : 1][EDGE ? KGS : 1][EDGE ? 4 : 1][EDGE ? 64 * 4 : 4];
  __shared__ float dump[EDGE ? 8 * DUMP : 1];
  __shared__ int bad_tile[2];  // per LDS stage: 1 + the last tile staged there with a non-finite Q or dO
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (EDGE && tid < 2) bad_tile[tid] = 0;
  const int kg = w & (KGS - 1);
  const int qg = QG == 1 ? 0 : (w >> 1) & 1;  // the half of every query tile that the wave takes
  const bool dk_role = w >= 4;  // wave-uniform
  const int nhb = N_heads * S_mb;
  const int kblk = blockIdx.x / nhb;  // earliest keys see the most queries: those blocks of every head go first
  const int head = (blockIdx.x % nhb) % N_heads, b = (blockIdx.x % nhb) / N_heads;
  const int h = N_heads * D;
  const size_t ld = 3 * (size_t)h;
  const bf16_t* base = qkv + (size_t)b * S_seq * ld + head * D;
  const bf16_t* dob = dctx + (size_t)b * S_seq * h + head * D;
  const float* lrow = lse + ((size_t)b * N_heads + head) * S_seq;
  const float* drow = delta + ((size_t)b * N_heads + head) * S_seq;
  const int k0 = kblk * KEYS, kw = k0 + 32 * kg, key = kw + (lane & 31);

  typename std::conditional<EDGE, FragAddrXor<D>, FragAddr<D>>::type fa;
  fa.init(lane);
  bf16x8 kvf[D / 16];  // this wave's K rows (dV role) or V rows (dK role): the B operand of its score-sized product
  load_rowfrags<D>(base + (size_t)(EDGE ? min(key, S_seq - 1) : key) * ld + (dk_role ? 2 * h : h), lane, kvf);
  const float c2 = scale * LOG2E;
  f32x16 acc[D / 32];  // dV (waves 0-3) or dK (waves 4-7), transposed: rows = head dims, column = key
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt) acc[dt] = zero16();

  const int jbeg = causal ? k0 / BLK : 0, nblk = EDGE ? (S_seq + BLK - 1) / BLK : S_seq / BLK;
  TileRegs<BLK, D, NTHR_DKV> qr, dor;
  float lnext = 0.f, dnext = 0.f;
  auto fetch = [&](int j) {
    const int i = j * BLK + tid;
    if constexpr (EDGE) {
      qr.load_edge(base + (size_t)j * BLK * ld, ld, tid, S_seq - j * BLK);
      dor.load_edge(dob + (size_t)j * BLK * h, h, tid, S_seq - j * BLK);
      // past the end: exp2(score - inf) = 0, no probability
      if (tid < BLK) { lnext = i < S_seq ? lrow[i] * LOG2E : INFINITY; dnext = i < S_seq ? drow[i] : 0.f; }
    } else {
      qr.load(base + (size_t)j * BLK * ld, ld, tid);
      dor.load(dob + (size_t)j * BLK * h, h, tid);
      if (tid < BLK) { lnext = lrow[i] * LOG2E; dnext = drow[i]; }
    }
  };
  auto note = [&](int j, int stage) {
    if (EDGE && (qr.non_finite() || dor.non_finite())) bad_tile[stage] = j + 1;
  };
  fetch(jbeg);
  if (EDGE) __syncthreads();  // bad_tile is clear
  qr.store(QOs[0][0], tid);
  dor.store(QOs[0][1], tid);
  note(jbeg, 0);
  if (tid < BLK) { stat_s[0][0][tid] = lnext; stat_s[0][1][tid] = dnext; }
  if (jbeg + 1 < nblk) fetch(jbeg + 1);
  __syncthreads();
  // Every wave passes the same barriers per query tile: one per hand-over of P and one at the end
  // (the other LDS stage is complete, this one may be overwritten).
  for (int j = jbeg; j < nblk; ++j) {
    const int cur = (j - jbeg) & 1;
    if constexpr (EDGE) fa.loop();
    const bf16_t* Qs = QOs[cur][0];
    const bf16_t* dOs = QOs[cur][1];
    const float* lse_s = stat_s[cur][0];
    const float* delta_s = stat_s[cur][1];
    if (j + 1 < nblk) {
      qr.store(QOs[cur ^ 1][0], tid);
      dor.store(QOs[cur ^ 1][1], tid);
      if (tid < BLK) { stat_s[cur ^ 1][0][tid] = lnext; stat_s[cur ^ 1][1][tid] = dnext; }
      note(j + 1, cur ^ 1);
    }
    if (j + 2 < nblk) fetch(j + 2);
    const int qb = j * BLK;
    // every query of the tile is before this pair's keys: nothing to add (the partner skips as well)
    const bool skip = (causal && qb + (QG == 1 ? BLK : 32 * qg + 32) - 1 < kw) || (EDGE && kw >= S_seq);
    const bool diag = causal && qb + 32 * qg < kw + 31;
    // Sub-tiles T0 .. T1-1 (32 queries each) go through the two stages together; every wave passes the
    // hand-over barrier between the stages, whether it has work or not.
    auto stages = [&](auto t0, auto t1) {
      constexpr int TC = decltype(t0)::value, NTT = decltype(t1)::value - TC;
      const int T0 = QG == 1 ? TC : qg;
      bf16x8 pb[NTT][2];
      f32x16 s[NTT];  // S, then P (dV role); dP, then dS (dK role)
#pragma unroll
      for (int u = 0; u < NTT; ++u) s[u] = zero16();
      if (!skip) {
        __builtin_amdgcn_sched_barrier(0);
        if (!dk_role) {
#pragma unroll
          for (int kk = 0; kk < D / 16; ++kk)
#pragma unroll
            for (int u = 0; u < NTT; ++u)
              s[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa.frag_k(Qs, 32 * (T0 + u), kk), kvf[kk], s[u], 0, 0, 0);
          mfma_lds_pipeline<NTT * (D / 16), 1, 4>();
          // P = exp(S / sqrt(d) - lse)
#pragma unroll
          for (int u = 0; u < NTT; ++u) {
            const int t = T0 + u;
#pragma unroll
            for (int r = 0; r < 16; ++r) s[u][r] = __builtin_amdgcn_exp2f(fmaf(s[u][r], c2, -lse_s[32 * t + acc_row(r, lane)]));
            if (diag) {
#pragma unroll
              for (int r = 0; r < 16; ++r)
                if (key > qb + 32 * t + acc_row(r, lane)) s[u][r] = 0.f;
            }
            if constexpr (EDGE) {
#pragma unroll
              for (int q4 = 0; q4 < 4; ++q4)
                *reinterpret_cast<f32x4*>(&Pf[t][kg][q4][lane * 4]) = f32x4{s[u][4 * q4], s[u][4 * q4 + 1], s[u][4 * q4 + 2], s[u][4 * q4 + 3]};
            } else {
              pb[u][0] = pack8(s[u], 0);
              pb[u][1] = pack8(s[u], 1);
              *reinterpret_cast<bf16x8*>(&Ps[t][kg][0][lane * 8]) = pb[u][0];
              *reinterpret_cast<bf16x8*>(&Ps[t][kg][1][lane * 8]) = pb[u][1];
            }
          }
        } else {
          // dP = dO V^T
#pragma unroll
          for (int kk = 0; kk < D / 16; ++kk)
#pragma unroll
            for (int u = 0; u < NTT; ++u)
              s[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa.frag_k(dOs, 32 * (T0 + u), kk), kvf[kk], s[u], 0, 0, 0);
          mfma_lds_pipeline<NTT * (D / 16), 1, 4>();
        }
      }
      __syncthreads();
      if constexpr (EDGE) {
        if (!skip) {
          if (dk_role) {
            // dS = P (dP - delta); masked pairs by selection (dP may be anything there), in a pass of its own: a condition at
            // every pair became a branch around its LDS reads, 16 waits in a row
            const bool mask = diag || qb + BLK > S_seq;
#pragma unroll
            for (int u = 0; u < NTT; ++u) {
              const int t = T0 + u;
#pragma unroll
              for (int q4 = 0; q4 < 4; ++q4) {
                const f32x4 p = *reinterpret_cast<const f32x4*>(&Pf[t][kg][q4][lane * 4]);
                const f32x4 dl = *reinterpret_cast<const f32x4*>(&delta_s[32 * t + acc_row(4 * q4, lane)]);
#pragma unroll
                for (int e = 0; e < 4; ++e) s[u][4 * q4 + e] = p[e] * (s[u][4 * q4 + e] - dl[e]);
              }
              if (mask) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                  const int i = qb + 32 * t + acc_row(r, lane), last = causal ? key : 0;
                  if (i < last || i >= S_seq) s[u][r] = 0.f;
                }
              }
            }
          }
          const bf16_t* tile = dk_role ? Qs : dOs;
          if (bad_tile[cur] == j + 1 || past_bf16(s)) {
            accumulate_allowed<D, NTT>(acc, s, T0, tile, dump + w * DUMP, lane, [&](int row) { return (!causal || key <= qb + row) && qb + row < S_seq; });
          } else {
#pragma unroll
            for (int u = 0; u < NTT; ++u) accumulate_split<D>(acc, s[u], tile, 32 * (T0 + u), fa);
          }
        }
        return;
      }
      if (!skip) {
        if (!dk_role) {
          // dV += dO^T P
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int u = 0; u < NTT; ++u)
#pragma unroll
            for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
              for (int dt = 0; dt < D / 32; ++dt)
                acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa.frag_t(dOs, 32 * (T0 + u) + 16 * k2, dt), pb[u][k2], acc[dt], 0, 0, 0);
          mfma_lds_pipeline<NTT * 2 * (D / 32), 2, 4>();
        } else {
          // dS = P (dP - delta) (the factor 1/sqrt(d) is applied once, to dK; masked entries of P are zero);  dK += Q^T dS
#pragma unroll
          for (int u = 0; u < NTT; ++u) {
            const int t = T0 + u;
            pb[u][0] = *reinterpret_cast<const bf16x8*>(&Ps[t][kg][0][lane * 8]);
            pb[u][1] = *reinterpret_cast<const bf16x8*>(&Ps[t][kg][1][lane * 8]);
#pragma unroll
            for (int r = 0; r < 16; ++r)
              s[u][r] = (float)pb[u][r >> 3][r & 7] * (s[u][r] - delta_s[32 * t + acc_row(r, lane)]);
            pb[u][0] = pack8(s[u], 0);
            pb[u][1] = pack8(s[u], 1);
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int u = 0; u < NTT; ++u)
#pragma unroll
            for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
              for (int dt = 0; dt < D / 32; ++dt)
                acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa.frag_t(Qs, 32 * (T0 + u) + 16 * k2, dt), pb[u][k2], acc[dt], 0, 0, 0);
          mfma_lds_pipeline<NTT * 2 * (D / 32), 2, 4>();
        }
      }
    };
    typedef std::integral_constant<int, 0> T_0;
    typedef std::integral_constant<int, 1> T_1;
    typedef std::integral_constant<int, 2> T_2;
    if constexpr (QG == 2) {
      stages(T_0{}, T_1{});
    } else if constexpr (D == 128 && !EDGE) {
      // both sub-tiles together: two independent accumulators in the score-sized products, one
      // hand-over barrier per tile (measured: 2 % faster than one sub-tile at a time at S_head 128,
      // 7 % slower at S_head 64)
      stages(T_0{}, T_2{});
    } else {
      stages(T_0{}, T_1{});
      stages(T_1{}, T_2{});
    }
    __syncthreads();
  }
  if constexpr (QG == 2) {
    // the second query group's sums, lane to lane (the tiles are free: the loop ended on a barrier)
    constexpr int NV = D / 2;
    static_assert(4 * NV * 64 * 4 <= sizeof(QOs), "the hand-over does not fit");
    float* hb = reinterpret_cast<float*>(&QOs[0][0][0]) + ((dk_role ? 2 : 0) + kg) * NV * 64 + lane;
    if (qg == 1) {
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) hb[(dt * 16 + r) * 64] = acc[dt][r];
    }
    __syncthreads();
    if (qg == 1) return;
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[dt][r] += hb[(dt * 16 + r) * 64];
  }
  if (EDGE && key >= S_seq) return;
  bf16_t* out = dqkv + ((size_t)b * S_seq + key) * ld + head * D;
  if (dk_role) store_rows<D>(acc, out + h, lane, scale);
  else store_rows<D>(acc, out + 2 * h, lane, 1.0f);
  if (!EDGE && colpart) {
    // row (b, key block) of the partial column sums of [dK | dV], [S_mb * S_seq / 128][2 N_heads * D]
    float* red = reinterpret_cast<float*>(&QOs[0][0][0]);
    wave_colsum<D>(acc, dk_role ? scale : 1.0f, red + (size_t)w * 4 * (D / 2), lane);
    __syncthreads();
    if (tid < 2 * D) {
      const int dv = tid / D, d = tid - dv * D;  // dK from waves 4-7, dV from waves 0-3
      colpart[((size_t)b * (S_seq / WG_ROWS) + kblk) * 2 * h + dv * h + head * D + d] = colsum_of<D>(red, dv ? 0 : 4, 4, d);
    }
  }
}

template <int D>
bf_status fwd_d(int S_mb, int S_seq, int N_heads, int causal, const void* qkv, void* ctx, float* lse, hipStream_t st, bool shared_chip) {
  const long blocks = (long)(S_seq / WG_ROWS) * N_heads * S_mb;
  const float scale = 1.0f / sqrtf((float)D);
  // Two key groups per workgroup halve the chain of key tiles of a row, which is the time of a launch that leaves compute
  // units idle (all of them but those of the longest rows, if causal).  Measured, one group / two on 64 rows / two on 128
  // rows, us: S_head 128, S_seq 2048 causal, 8 heads 50 / 45 / 42, 16 heads 52 / 53 / 44, 32 heads 68 / 106 / 57, 64 heads
  // 88 / 206 / 111; bidirectional, 16 heads 53 / 87 / 49, 32 heads 76 / 199 / 93; S_seq 512, 16 heads 16.5 / 14.9 / 16.2;
  // S_head 64, S_seq 2048 causal, 16 heads 36 / 30 / 27, 32 heads 46 / 43 / 35, 64 heads 62 / 85 / 76.  Shorter causal rows hide
  // less: S_head 128, one group / two on 128 rows, S_seq 1280 at 480 blocks 38.0 / 40.4, 1152 at 432 34.5 / 36.1, 1024 at 384
  // 30.9 / 31.7.  Beside another stream's kernels, which fill the units that the longest rows leave (a 2048-wide step on two
  // chains, 256 blocks causal: 36.2 ms with two groups here, 35.5 with one): up to 128 blocks.
  const long two_groups = shared_chip ? 128 : !causal ? 256 : D == 128 && S_seq < 1792 ? 320 : 512;
  if (S_seq >= 1024 && blocks <= two_groups) {
    attn_fwd_general_kernel<D, 128, false, 2><<<(unsigned)blocks, 512, 0, st>>>((const bf16_t*)qkv, (bf16_t*)ctx, lse, S_seq, N_heads, S_mb, causal, scale);
  } else if (S_seq >= 256 && S_seq < 1024 && blocks <= 128) {
    attn_fwd_general_kernel<D, 64, false, 2><<<(unsigned)(2 * blocks), 256, 0, st>>>((const bf16_t*)qkv, (bf16_t*)ctx, lse, S_seq, N_heads, S_mb, causal, scale);
  } else
  // the 256-query form when there are enough (head, block) pairs to give every compute unit one
  if (S_seq % 256 == 0 && (long)(S_seq / 256) * N_heads * S_mb >= 256) {
    const unsigned grid = (unsigned)(S_seq / 256) * N_heads * S_mb;
    attn_fwd_kernel<D, 256><<<grid, 512, 0, st>>>((const bf16_t*)qkv, (bf16_t*)ctx, lse, S_seq, N_heads, S_mb, causal, 1.0f / sqrtf((float)D));
  } else {
    const unsigned grid = (unsigned)(S_seq / 128) * N_heads * S_mb;
    attn_fwd_kernel<D, 128><<<grid, 256, 0, st>>>((const bf16_t*)qkv, (bf16_t*)ctx, lse, S_seq, N_heads, S_mb, causal, 1.0f / sqrtf((float)D));
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_error("attention_fwd_mfma launch failed: %s", hipGetErrorString(e)); return BF_EDEVICE; }
  return BF_OK;
}

// out[r][n] = sum of rows fold * r .. fold * r + fold - 1 of in, in order
__global__ __launch_bounds__(64) void fold_rows_kernel(const float* __restrict__ in, float* __restrict__ out, int fold, int h) {
  const int n = blockIdx.x * 64 + threadIdx.x;
  if (n >= h) return;
  const float* p = in + (size_t)blockIdx.y * fold * h + n;
  float t = p[0];
  for (int k = 1; k < fold; ++k) t += p[(size_t)k * h];
  out[(size_t)blockIdx.y * h + n] = t;
}

template <int D>
bf_status bwd_d(int S_mb, int S_seq, int N_heads, int causal, const void* qkv, const void* ctx, const float* lse,
                const void* dctx, void* dqkv, float* delta, float* part, hipStream_t st, bool shared_chip) {
  const float scale = 1.0f / sqrtf((float)D);
  const unsigned grid = (unsigned)(S_seq / WG_ROWS) * N_heads * S_mb;
  // partial column sums: dQ's rows first, then those of [dK | dV]
  float* part_kv = part ? part + attention_bwd_mfma_part_q_rows(S_mb, S_seq) * (size_t)N_heads * D : nullptr;
  // Two key groups on 64 rows, as in the forward pass (S_head 128, S_seq 2048 causal, 8 / 16 / 32 heads: 81 -> 53, 83 -> 66,
  // 88 -> 125 us; bidirectional, 8 / 16 heads 81 -> 53, 84 -> 104; S_head 64, causal, 16 / 32 heads 47 -> 31, 50 -> 49; on 128
  // rows it spills).  Its partial column sums, one row per 64 queries, go where those of [dK | dV] will be and are folded
  // into the rows per 256 (or 128) queries that the scratch has (4 us).
  // Beside another stream's kernels the longest rows' units are not the only busy ones, and from 257 workgroups on the
  // second group costs more than it hides (a 2048-wide step on two chains: attention backward 8.9 -> 9.9 ms, step 36.5 -> 37.6, with two).
  // Nor does it pay on rows of two tiles then (S_seq 256, 100 heads of 128, causal: 39.4 -> 43.3 us; 384, 80 heads: 47.2 / 47.5).
  if (S_seq >= (grid > 128 ? 384 : 256) && 2 * (long)grid <= (causal && !shared_chip ? 512 : 256)) {
    attn_bwd_dq_general_kernel<D, 64, false, 2><<<grid * 2, 256, 0, st>>>((const bf16_t*)qkv, (const bf16_t*)ctx, (const bf16_t*)dctx, lse, delta, (bf16_t*)dqkv, S_seq, N_heads, S_mb, causal, scale, part_kv);
    if (part) {
      const int h = N_heads * D, rows = (int)attention_bwd_mfma_part_q_rows(S_mb, S_seq);
      fold_rows_kernel<<<dim3((h + 63) / 64, rows), 64, 0, st>>>(part_kv, part, S_mb * (S_seq / 64) / rows, h);
    }
  } else if (S_seq % 256 == 0)  // measured faster than the 128-query form also on grids that do not fill the chip
    attn_bwd_dq_kernel<D, 256><<<grid / 2, 512, 0, st>>>((const bf16_t*)qkv, (const bf16_t*)ctx, (const bf16_t*)dctx, lse, delta, (bf16_t*)dqkv, S_seq, N_heads, S_mb, causal, scale, part);
  else
    attn_bwd_dq_kernel<D, 128><<<grid, NTHR, 0, st>>>((const bf16_t*)qkv, (const bf16_t*)ctx, (const bf16_t*)dctx, lse, delta, (bf16_t*)dqkv, S_seq, N_heads, S_mb, causal, scale, part);
  if (attention_bwd_dkv_wide_supported(S_mb, S_seq, N_heads, D) && attention_bwd_dkv_wide_better(S_mb, S_seq, N_heads, D, causal)) {
    const bf_status r = attention_bwd_dkv_wide(S_mb, S_seq, N_heads, D, causal, qkv, lse, dctx, dqkv, delta, part_kv, st);
    if (r != BF_OK) return r;
  } else {
    attn_bwd_dkv_kernel<D><<<grid, NTHR_DKV, 0, st>>>((const bf16_t*)qkv, (const bf16_t*)dctx, lse, delta, (bf16_t*)dqkv, S_seq, N_heads, S_mb, causal, scale, part_kv);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_error("attention_bwd_mfma launch failed: %s", hipGetErrorString(e)); return BF_EDEVICE; }
  return BF_OK;
}

// The EDGE forms, the last block of rows partly empty; no partial column sums.  Two key groups for launches of few rows,
// as in fwd_d and bwd_d (S_head 128 on 64 rows: on 128 they spill).  Forward, one group / two, us: S_head 128, causal, 1000
// tokens, 16 heads 47 / 34, twice that 51 / 48 (bidirectional 51 / 70), 2 x 1900 tokens 90 / 126; S_head 64, 1900 tokens, 16
// heads 51 / 36, 4 x 1000 tokens 33 / 31.  Short rows hide less: S_head 64, causal, 257 tokens at 300 blocks 12.0 / 15.9, 400 at
// 400 18.0 / 21.0, 600 at 500 25.2 / 27.2, 700 at 480 25.4 / 26.4, 900 at 512 level; S_head 128, causal, 257 tokens at 240 blocks
// 18.2 / 19.7, 300 at 240 19.6 / 19.8.
template <int D>
bf_status fwd_edge(int S_mb, int S_seq, int N_heads, int causal, const void* qkv, void* ctx, float* lse, hipStream_t st) {
  const long blocks = (long)((S_seq + 127) / 128) * N_heads * S_mb;
  const float scale = 1.0f / sqrtf((float)D);
  constexpr int EDGE_ROWS = D == 64 ? 128 : 64;
  const long two_groups = D == 64 ? (causal && S_seq >= 768 ? 512 : 256) : !causal ? 128 : S_seq >= 384 ? 256 : 192;
  if (S_seq > 256 && blocks <= two_groups)
    attn_fwd_general_kernel<D, EDGE_ROWS, true, 2><<<(unsigned)((S_seq + EDGE_ROWS - 1) / EDGE_ROWS) * N_heads * S_mb, 4 * EDGE_ROWS, 0, st>>>((const bf16_t*)qkv, (bf16_t*)ctx, lse, S_seq, N_heads, S_mb, causal, scale);
  else
    attn_fwd_general_kernel<D, 128, true, 1><<<(unsigned)blocks, 256, 0, st>>>((const bf16_t*)qkv, (bf16_t*)ctx, lse, S_seq, N_heads, S_mb, causal, scale);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_error("attention_fwd_mfma launch failed: %s", hipGetErrorString(e)); return BF_EDEVICE; }
  return BF_OK;
}

template <int D>
bf_status bwd_edge(int S_mb, int S_seq, int N_heads, int causal, const void* qkv, const void* ctx, const float* lse,
                   const void* dctx, void* dqkv, float* delta, hipStream_t st) {
  const float scale = 1.0f / sqrtf((float)D);
  const unsigned grid = (unsigned)((S_seq + 127) / 128) * N_heads * S_mb;
  // Two key groups up to 256 causal blocks of 128 rows; up to 128 bidirectional ones, and causal ones of short rows at S_head
  // 128.  One group / two, backward, us: S_head 128, causal, 256 blocks, 1000 tokens 156.8 / 147.7, 900 145.2 / 138.0, 400
  // 3 % more with two, 200 11 %; 300 to 512 blocks 4 to 10 %; bidirectional, 129 to 256 blocks 7 to 20 %.
  if (S_seq > 128 && 2 * (long)grid <= (causal && (D == 64 || S_seq >= 900) ? 512 : 256))
    attn_bwd_dq_general_kernel<D, 64, true, 2><<<(unsigned)((S_seq + 63) / 64) * N_heads * S_mb, 256, 0, st>>>((const bf16_t*)qkv, (const bf16_t*)ctx, (const bf16_t*)dctx, lse, delta, (bf16_t*)dqkv, S_seq, N_heads, S_mb, causal, scale, nullptr);
  else
    attn_bwd_dq_general_kernel<D, 128, true, 1><<<grid, NTHR, 0, st>>>((const bf16_t*)qkv, (const bf16_t*)ctx, (const bf16_t*)dctx, lse, delta, (bf16_t*)dqkv, S_seq, N_heads, S_mb, causal, scale, nullptr);
  // Two query groups (64 keys a workgroup, half of every query tile each) where the chip does not fill: a workgroup has a compute
  // unit to itself and takes 0.52 (S_head 128) or 0.6 (64) of the time of 128 keys with one group, so for bidirectional
  // launches the rounds of 256 decide.  Causal ones last as long as their longest key block, twice the mean, until the other
  // blocks' tiles come to more than that per compute unit (`fill`, in longest blocks), and past that the second group only costs;
  // long rows, with many blocks to even out, gain a little longer.  Backward, one group / two, us, S_head 128: causal,
  // 1000 tokens, 128 blocks of 128 keys 121 / 81 (fill 0.28), 256 136 / 104 (0.56), 384 148 / 146 (0.84), 896 355 / 350 (2.0), 1024 388 / 399;
  // 300 tokens, 192 blocks 62 / 48 (0.45), 384 79.7 / 83.5 (0.9), 200 tokens, 256 blocks 58 / 54 (0.75), 512 97.6 / 102.6 (1.5), 65 tokens, 128
  // 34 / 31 (0.5), 256 38.4 / 40.2 (1.0); bidirectional, 1000 tokens, 128 blocks 123 / 85, 256 (two rounds) 152 / 154, 384 (three for two)
  // 291 / 254, 500 tokens, 192 blocks 84 / 86.  S_head 64: causal, 700 tokens, 192 blocks 58 / 46 (0.41), 288 67 / 64 (0.61), 384 69 / 74
  // (0.82), 2000 tokens, 256 blocks 18 % less (0.53), 320 2 % less (0.66), 384 6 % more (0.8); bidirectional, 128
  // blocks 74 / 58, 192 65 / 75, 384 in three rounds for two 115 / 112, 576 in five for three 170 / 179.
  const long heads = (long)N_heads * S_mb, n = (S_seq + 63) / 64, blocks = (S_seq + 127) / 128;
  const long grid2 = n * heads, rounds1 = ((long)grid + 255) / 256, rounds2 = (grid2 + 255) / 256;
  const double fill = (double)heads * (double)(blocks * n - blocks * (blocks - 1)) / (256.0 * (double)n);
  const double fill_max = D == 64 ? 0.68 : std::max(0.85, std::min(2.0, (double)n / 8));
  const bool two_query_groups = causal ? fill <= fill_max : D == 128 ? rounds2 < 2 * rounds1 : 5 * rounds2 <= 8 * rounds1;
  if (two_query_groups && grid2 < (1l << 31))
    attn_bwd_dkv_kernel<D, true, 2><<<(unsigned)grid2, NTHR_DKV, 0, st>>>((const bf16_t*)qkv, (const bf16_t*)dctx, lse, delta, (bf16_t*)dqkv, S_seq, N_heads, S_mb, causal, scale, nullptr);
  else
    attn_bwd_dkv_kernel<D, true><<<grid, NTHR_DKV, 0, st>>>((const bf16_t*)qkv, (const bf16_t*)dctx, lse, delta, (bf16_t*)dqkv, S_seq, N_heads, S_mb, causal, scale, nullptr);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_error("attention_bwd_mfma launch failed: %s", hipGetErrorString(e)); return BF_EDEVICE; }
  return BF_OK;
}

bool args_ok(int S_mb, int S_seq, int N_heads, int S_head, const void* a, const void* b2) {
  if (!attention_mfma_supported(S_seq, S_head)) { set_error("attention_mfma: needs S_head 64 or 128 and S_seq a multiple of 128"); return false; }
  if (S_mb < 1 || N_heads < 1 || S_mb > 65535 || N_heads > 65535) { set_error("attention_mfma: bad S_mb / N_heads"); return false; }
  if (((uintptr_t)a | (uintptr_t)b2) & 15) { set_error("attention_mfma: tensors must be 16-byte aligned"); return false; }
  return true;
}

}  // namespace

bool attention_mfma_supported(int S_seq, int S_head) {
  return (S_head == 64 || S_head == 128) && S_seq >= WG_ROWS && S_seq % WG_ROWS == 0;
}

bool attention_mfma_edge_supported(int S_mb, int S_seq, int N_heads, int S_head) {
  return (S_head == 64 || S_head == 128) && S_seq >= 1 && S_seq <= 4096 && S_mb >= 1 && N_heads >= 1 && S_mb <= 65535 && N_heads <= 65535 &&
         (long)((S_seq + 127) / 128) * N_heads * S_mb < (1l << 31);
}

bf_status attention_fwd_mfma_edge(int S_mb, int S_seq, int N_heads, int S_head, int causal, const void* qkv, void* ctx, float* lse,
                                  hipStream_t st) {
  return S_head == 128 ? fwd_edge<128>(S_mb, S_seq, N_heads, causal, qkv, ctx, lse, st) : fwd_edge<64>(S_mb, S_seq, N_heads, causal, qkv, ctx, lse, st);
}

bf_status attention_bwd_mfma_edge(int S_mb, int S_seq, int N_heads, int S_head, int causal, const void* qkv, const void* ctx,
                                  const float* lse, const void* dctx, void* dqkv, float* delta, hipStream_t st) {
  return S_head == 128 ? bwd_edge<128>(S_mb, S_seq, N_heads, causal, qkv, ctx, lse, dctx, dqkv, delta, st)
                       : bwd_edge<64>(S_mb, S_seq, N_heads, causal, qkv, ctx, lse, dctx, dqkv, delta, st);
}

bf_status attention_fwd_mfma(int S_mb, int S_seq, int N_heads, int S_head, int causal, const void* qkv, void* ctx,
                             float* lse, hipStream_t st, bool shared_chip) {
  if (!args_ok(S_mb, S_seq, N_heads, S_head, qkv, ctx)) return BF_EINVAL;
  if (S_head == 128) return fwd_d<128>(S_mb, S_seq, N_heads, causal, qkv, ctx, lse, st, shared_chip);
  return fwd_d<64>(S_mb, S_seq, N_heads, causal, qkv, ctx, lse, st, shared_chip);
}

// Rows of partial column sums the two backward kernels leave: one per (micro-batch sequence, query block) for dQ
// and one per (sequence, block of 128 keys) for [dK | dV].
size_t attention_bwd_mfma_part_q_rows(int S_mb, int S_seq) { return (size_t)S_mb * (S_seq / (S_seq % 256 == 0 ? 256 : WG_ROWS)); }
size_t attention_bwd_mfma_part_kv_rows(int S_mb, int S_seq) { return (size_t)S_mb * (S_seq / WG_ROWS); }

bf_status attention_bwd_mfma(int S_mb, int S_seq, int N_heads, int S_head, int causal, const void* qkv, const void* ctx,
                             const float* lse, const void* dctx, void* dqkv, float* delta, hipStream_t st, float* part, bool shared_chip) {
  if (!args_ok(S_mb, S_seq, N_heads, S_head, qkv, dqkv) || !args_ok(S_mb, S_seq, N_heads, S_head, ctx, dctx)) return BF_EINVAL;
  if (S_head == 128) return bwd_d<128>(S_mb, S_seq, N_heads, causal, qkv, ctx, lse, dctx, dqkv, delta, part, st, shared_chip);
  return bwd_d<64>(S_mb, S_seq, N_heads, causal, qkv, ctx, lse, dctx, dqkv, delta, part, st, shared_chip);
}

}  // namespace bf
