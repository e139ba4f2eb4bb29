// Attention on the fp32 matrix instructions, forward and backward: fp32 mode, and the bf16 shapes that the bf16 kernels
// do not take.  Any S_seq up to 4096, head sizes up to 128, probabilities and sums in fp32 throughout.
//
// v_mfma_f32_16x16x4_f32 contracts its four k one after the other with one rounding each, so a product contracted in
// ascending order is the chain of fused multiply-adds that the plain kernels (attention_plain.hip) compute; everything
// else here is done in their order too, so the results are the same bits, which the tests check.
//
// A workgroup of four waves owns 16 RT rows (queries; in the dK / dV pass keys) of one head and walks the other side in
// tiles of 64.  In the score-sized products wave w takes 16 of the 64 columns, in the head-sized ones every fourth 16
// head dimensions.  Lane l holds row / column l % 16 and k = 4 s + l / 16 in step s.  The row pitches of the LDS tiles are
// 4 words past a multiple of 64: 16 rows x 4 consecutive k are 64 different banks.
//
// A zero probability times an infinity is a NaN in a matrix instruction, but a masked pair must not touch its row: tiles
// that reach past the mask are searched for non-finite values as they are staged and, if there are any, contracted
// element by element over the allowed pairs only.
//
// Small launches are bound by latency and the length of the chains, large ones by the matrix pipeline and the tiles' reads.
// Forward / dQ / dK dV, plain kernels against these: fp32, 4 heads of 64, S_seq 128: 15 / 15 / 23 -> 8 / 9 / 11 us; bf16, 2
// sequences of 1000, 16 heads of 128, causal: 787 / 1535 / 1925 -> 422 / 395 / 516 us.
#include <type_traits>

#include "common.h"

namespace bf {

namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

constexpr int NT = 256;   // four waves
constexpr int BLK = 64;   // rows of a streamed tile
constexpr int PLD = BLK + 4;

__device__ __forceinline__ float wsum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wmax(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ bool non_finite(float v) { return (__builtin_bit_cast(uint32_t, v) & 0x7f800000u) == 0x7f800000u; }

template <typename T, int VEC>
struct alignas(sizeof(T) * VEC) Pack { T v[VEC]; };

// ROWS rows of head dimensions (DP >= d columns, zeros past d and past the last valid row): global -> registers -> LDS
template <typename T, int VEC, int ROWS, int DP>
struct Rows {
  static constexpr int LD = DP + 4, CPR = DP / VEC, CH = ROWS * CPR / NT;
  static_assert(ROWS * CPR % NT == 0, "the chunks must divide among the threads");
  Pack<T, VEC> v[CH];
  __device__ __forceinline__ void load(const T* __restrict__ g, size_t ld, int valid, int d, int tid) {
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int c = tid + i * NT, row = c / CPR, col = c % CPR * VEC;
      if (row < valid && col < d) {
        v[i] = *reinterpret_cast<const Pack<T, VEC>*>(g + (size_t)row * ld + col);
      } else {
#pragma unroll
        for (int j = 0; j < VEC; ++j) v[i].v[j] = (T)0.f;
      }
    }
  }
  // returns whether one of the thread's values is an infinity or a NaN
  __device__ __forceinline__ bool store(float* lds, int tid) const {
    bool bad = false;
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int c = tid + i * NT, row = c / CPR, col = c % CPR * VEC;
#pragma unroll
      for (int j = 0; j < VEC; ++j) {
        const float f = (float)v[i].v[j];
        bad |= non_finite(f);
        lds[row * LD + col + j] = f;
      }
    }
    return bad;
  }
};

__device__ __forceinline__ f32x4 mma(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// out[rt] = rows of `a` (16 rt ..) times the 16 rows of `b`, contracted along the head dimensions
template <int RT, int DP>
__device__ __forceinline__ void scores(const float* a, const float* b, int lane, f32x4 (&out)[RT]) {
  constexpr int LD = DP + 4;
  const int q = lane >> 4, l16 = lane & 15;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) out[rt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
  for (int s = 0; s < DP / 4; ++s) {
    const float bv = b[l16 * LD + 4 * s + q];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) out[rt] = mma(a[(rt * 16 + l16) * LD + 4 * s + q], bv, out[rt]);
  }
}

// acc[rt][k] += p (16 RT rows x 64, pitch ldp) times the 64 rows of `b`, for the head dimensions 16 (w + 4 k) + lane % 16.
// bad: the tile holds non-finite values; then only the pairs allowed(row, column) are added, in the same order.
template <int RT, int DP, typename F>
__device__ __forceinline__ void accumulate(const float* p, int ldp, const float* b, int w, int lane, bool bad, F allowed,
                                           f32x4 (&acc)[RT][DP / 64]) {
  constexpr int LD = DP + 4;
  const int q = lane >> 4, l16 = lane & 15;
  if (!bad) {
#pragma unroll 4
    for (int s = 0; s < BLK / 4; ++s) {
      float av[RT];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) av[rt] = p[(rt * 16 + l16) * ldp + 4 * s + q];
#pragma unroll
      for (int k = 0; k < DP / 64; ++k) {
        const float bv = b[(4 * s + q) * LD + (w + 4 * k) * 16 + l16];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) acc[rt][k] = mma(av[rt], bv, acc[rt][k]);
      }
    }
  } else {
    for (int j = 0; j < BLK; ++j)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = rt * 16 + q * 4 + r;
          if (!allowed(row, j)) continue;
#pragma unroll
          for (int k = 0; k < DP / 64; ++k) acc[rt][k][r] = fmaf(p[row * ldp + j], b[j * LD + (w + 4 * k) * 16 + l16], acc[rt][k][r]);
        }
  }
}

// f(row, head dimension, rt, k, r) for the lane's elements of an accumulator set that lie inside the matrix
template <int RT, int DP, typename F>
__device__ __forceinline__ void each_out(int w, int lane, int rows, int d, F f) {
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int k = 0; k < DP / 64; ++k)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = rt * 16 + (lane >> 4) * 4 + r, c = (w + 4 * k) * 16 + (lane & 15);
        if (row < rows && c < d) f(row, c, rt, k, r);
      }
}

// The scores of the workgroup's rows stay in LDS between the products (dynamic part, 16 RT x (S rounded up to 64, + 4)):
// the softmax needs a row's maximum before the first exponential, and the plain order of its sum.
template <typename T, int VEC, int RT, int DP>
__global__ __launch_bounds__(NT) void attn_fwd_f32_kernel(const T* __restrict__ qkv, T* __restrict__ ctx, float* __restrict__ lse, int S_seq,
                                                          int N_heads, int d, int causal, float scale) {
  typedef Rows<T, VEC, BLK, DP> Tile;
  typedef Rows<T, VEC, 16 * RT, DP> Own;
  extern __shared__ __attribute__((aligned(16))) float sc[];
  __shared__ __attribute__((aligned(16))) float Qs[16 * RT * Own::LD], Ks[BLK * Tile::LD];
  __shared__ float inv_s[16 * RT];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int i0 = blockIdx.x * 16 * RT, head = blockIdx.y, b = blockIdx.z, h = N_heads * d;
  const int rows = min(16 * RT, S_seq - i0), jmax = causal ? i0 + rows : S_seq, nt = (jmax + BLK - 1) / BLK;
  const int lds_s = (S_seq + BLK - 1) / BLK * BLK + 4;
  const size_t ld = 3 * (size_t)h;
  const T* base = qkv + (size_t)b * S_seq * ld + head * d;
  {
    Own q;
    q.load(base + (size_t)i0 * ld, ld, rows, d, tid);
    q.store(Qs, tid);
  }
  Tile t;
  t.load(base + h, ld, S_seq, d, tid);
  for (int j = 0; j < nt; ++j) {
    t.store(Ks, tid);
    __syncthreads();
    if (j + 1 < nt) t.load(base + (size_t)(j + 1) * BLK * ld + h, ld, S_seq - (j + 1) * BLK, d, tid);
    else t.load(base + 2 * h, ld, S_seq, d, tid);  // the first tile of V
    f32x4 s[RT];
    scores<RT, DP>(Qs, Ks + w * 16 * Tile::LD, lane, s);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int r = 0; r < 4; ++r) sc[(rt * 16 + (lane >> 4) * 4 + r) * lds_s + j * BLK + w * 16 + (lane & 15)] = s[rt][r] * scale;
    __syncthreads();
  }
  // softmax of a row by one wave: columns lane, lane + 64, ...
  for (int row = w; row < 16 * RT; row += 4) {
    float* sr = sc + row * lds_s;
    const int jend = row >= rows ? 0 : causal ? i0 + row + 1 : S_seq;
    float mx = -INFINITY;
    for (int j = lane; j < jend; j += 64) mx = fmaxf(mx, sr[j]);
    mx = wmax(mx);
    float sum = 0.f;
    for (int j = lane; j < nt * BLK; j += 64) {
      float e = 0.f;
      if (j < jend) {
        e = expf(sr[j] - mx);
        sum += e;
      }
      sr[j] = e;
    }
    sum = wsum(sum);
    if (lane == 0) {
      inv_s[row] = 1.0f / sum;
      if (row < rows) lse[((size_t)b * N_heads + head) * S_seq + i0 + row] = mx + logf(sum);
    }
  }
  f32x4 acc[RT][DP / 64] = {};
  for (int j = 0; j < nt; ++j) {
    const bool mine = t.store(Ks, tid);
    const int jb = j * BLK;
    const bool bad = __syncthreads_or(mine && causal && jb + BLK - 1 > i0);
    if (j + 1 < nt) t.load(base + (size_t)(j + 1) * BLK * ld + 2 * h, ld, S_seq - (j + 1) * BLK, d, tid);
    accumulate<RT, DP>(sc + jb, lds_s, Ks, w, lane, bad, [&](int row, int c) { return jb + c <= i0 + row; }, acc);
    __syncthreads();
  }
  each_out<RT, DP>(w, lane, rows, d, [&](int row, int c, int rt, int k, int r) {
    ctx[((size_t)b * S_seq + i0 + row) * h + head * d + c] = (T)(acc[rt][k][r] * inv_s[row]);
  });
}

template <typename T, int VEC, int RT, int DP>
__global__ __launch_bounds__(NT) void attn_bwd_dq_f32_kernel(const T* __restrict__ qkv, const T* __restrict__ dctx, const float* __restrict__ lse,
                                                             const float* __restrict__ delta, T* __restrict__ dqkv, int S_seq, int N_heads,
                                                             int d, int causal, float scale) {
  typedef Rows<T, VEC, BLK, DP> Tile;
  typedef Rows<T, VEC, 16 * RT, DP> Own;
  __shared__ __attribute__((aligned(16))) float Qs[16 * RT * Own::LD], Os[16 * RT * Own::LD], Ks[BLK * Tile::LD], Vs[BLK * Tile::LD];
  __shared__ float ds[16 * RT * PLD];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int i0 = blockIdx.x * 16 * RT, head = blockIdx.y, b = blockIdx.z, h = N_heads * d;
  const int rows = min(16 * RT, S_seq - i0), jmax = causal ? i0 + rows : S_seq, nt = (jmax + BLK - 1) / BLK;
  const size_t ld = 3 * (size_t)h;
  const T* base = qkv + (size_t)b * S_seq * ld + head * d;
  {
    Own q;
    q.load(base + (size_t)i0 * ld, ld, rows, d, tid);
    q.store(Qs, tid);
    q.load(dctx + ((size_t)b * S_seq + i0) * h + head * d, h, rows, d, tid);
    q.store(Os, tid);
  }
  float l[RT][4], dl[RT][4];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = rt * 16 + (lane >> 4) * 4 + r;
      const size_t st = ((size_t)b * N_heads + head) * S_seq + i0 + row;
      l[rt][r] = row < rows ? lse[st] : 0.f;
      dl[rt][r] = row < rows ? delta[st] : 0.f;
    }
  f32x4 acc[RT][DP / 64] = {};
  Tile tk, tv;
  tk.load(base + h, ld, S_seq, d, tid);
  tv.load(base + 2 * h, ld, S_seq, d, tid);
  for (int j = 0; j < nt; ++j) {
    const int jb = j * BLK;
    const bool mine = tk.store(Ks, tid);
    tv.store(Vs, tid);
    const bool bad = __syncthreads_or(mine && causal && jb + BLK - 1 > i0);
    if (j + 1 < nt) {
      tk.load(base + (size_t)(jb + BLK) * ld + h, ld, S_seq - jb - BLK, d, tid);
      tv.load(base + (size_t)(jb + BLK) * ld + 2 * h, ld, S_seq - jb - BLK, d, tid);
    }
    f32x4 s[RT], dp[RT];
    scores<RT, DP>(Qs, Ks + w * 16 * Tile::LD, lane, s);
    scores<RT, DP>(Os, Vs + w * 16 * Tile::LD, lane, dp);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = rt * 16 + (lane >> 4) * 4 + r, c = w * 16 + (lane & 15);
        const float p = expf(s[rt][r] * scale - l[rt][r]);
        const float v = p * (dp[rt][r] - dl[rt][r]) * scale;
        ds[row * PLD + c] = row < rows && jb + c < S_seq && !(causal && jb + c > i0 + row) ? v : 0.f;
      }
    __syncthreads();
    accumulate<RT, DP>(ds, PLD, Ks, w, lane, bad, [&](int row, int c) { return jb + c <= i0 + row; }, acc);
    __syncthreads();
  }
  each_out<RT, DP>(w, lane, rows, d, [&](int row, int c, int rt, int k, int r) {
    dqkv[((size_t)b * S_seq + i0 + row) * ld + head * d + c] = (T)acc[rt][k][r];
  });
}

// Rows are keys here, the streamed tiles queries; causal: from the tile of the first key on.
template <typename T, int VEC, int RT, int DP>
__global__ __launch_bounds__(NT) void attn_bwd_dkv_f32_kernel(const T* __restrict__ qkv, const T* __restrict__ dctx, const float* __restrict__ lse,
                                                              const float* __restrict__ delta, T* __restrict__ dqkv, int S_seq, int N_heads,
                                                              int d, int causal, float scale) {
  typedef Rows<T, VEC, BLK, DP> Tile;
  typedef Rows<T, VEC, 16 * RT, DP> Own;
  __shared__ __attribute__((aligned(16))) float Ks[16 * RT * Own::LD], Vs[16 * RT * Own::LD], Qs[BLK * Tile::LD], Os[BLK * Tile::LD];
  __shared__ float ps[16 * RT * PLD], ds[16 * RT * PLD];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int j0 = blockIdx.x * 16 * RT, head = blockIdx.y, b = blockIdx.z, h = N_heads * d;
  const int rows = min(16 * RT, S_seq - j0), t0 = causal ? j0 / BLK : 0, nt = (S_seq + BLK - 1) / BLK;
  const size_t ld = 3 * (size_t)h;
  const T* base = qkv + (size_t)b * S_seq * ld + head * d;
  const T* dob = dctx + (size_t)b * S_seq * h + head * d;
  const float* lrow = lse + ((size_t)b * N_heads + head) * S_seq;
  const float* drow = delta + ((size_t)b * N_heads + head) * S_seq;
  {
    Own k;
    k.load(base + (size_t)j0 * ld + h, ld, rows, d, tid);
    k.store(Ks, tid);
    k.load(base + (size_t)j0 * ld + 2 * h, ld, rows, d, tid);
    k.store(Vs, tid);
  }
  f32x4 dk[RT][DP / 64] = {}, dv[RT][DP / 64] = {};
  Tile tq, to;
  tq.load(base + (size_t)t0 * BLK * ld, ld, S_seq - t0 * BLK, d, tid);
  to.load(dob + (size_t)t0 * BLK * h, h, S_seq - t0 * BLK, d, tid);
  for (int t = t0; t < nt; ++t) {
    const int ib = t * BLK, i = ib + w * 16 + (lane & 15);
    const bool bad_q = tq.store(Qs, tid), bad_o = to.store(Os, tid);
    const bool edge = causal && ib < j0 + 16 * RT - 1;
    const int bad = __syncthreads_or(edge && (bad_q || bad_o));
    const float li = i < S_seq ? lrow[i] : 0.f, di = i < S_seq ? drow[i] : 0.f;
    if (t + 1 < nt) {
      tq.load(base + (size_t)(ib + BLK) * ld, ld, S_seq - ib - BLK, d, tid);
      to.load(dob + (size_t)(ib + BLK) * h, h, S_seq - ib - BLK, d, tid);
    }
    f32x4 s[RT], dp[RT];
    scores<RT, DP>(Ks, Qs + w * 16 * Tile::LD, lane, s);
    scores<RT, DP>(Vs, Os + w * 16 * Tile::LD, lane, dp);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = rt * 16 + (lane >> 4) * 4 + r, c = w * 16 + (lane & 15);
        const bool ok = i < S_seq && row < rows && !(causal && i < j0 + row);
        const float p = expf(s[rt][r] * scale - li);
        const float v = p * (dp[rt][r] - di) * scale;
        ps[row * PLD + c] = ok ? p : 0.f;
        ds[row * PLD + c] = ok ? v : 0.f;
      }
    __syncthreads();
    auto allowed = [&](int row, int c) { return ib + c >= j0 + row && ib + c < S_seq; };
    accumulate<RT, DP>(ds, PLD, Qs, w, lane, bad, allowed, dk);
    accumulate<RT, DP>(ps, PLD, Os, w, lane, bad, allowed, dv);
    __syncthreads();
  }
  each_out<RT, DP>(w, lane, rows, d, [&](int row, int c, int rt, int k, int r) {
    T* o = dqkv + ((size_t)b * S_seq + j0 + row) * ld + head * d + c;
    o[h] = (T)dk[rt][k][r];
    o[2 * h] = (T)dv[rt][k][r];
  });
}

constexpr size_t LDS_MAX = 160 * 1024;

// bytes of LDS of the forward kernel: its rows, a tile, the scores
size_t fwd_scores_bytes(int RT, int S_seq) { return (size_t)16 * RT * ((S_seq + BLK - 1) / BLK * BLK + 4) * sizeof(float); }
size_t fwd_fixed_bytes(int RT, int DP) { return ((size_t)(16 * RT + BLK) * (DP + 4) + 16 * RT) * sizeof(float) + 64; }

// 32 rows per workgroup read the other side half as often; 16 where 32 would leave compute units without a workgroup
// (or the forward pass without room for the scores).
int row_tiles(int S_mb, int S_seq, int N_heads) { return (long)((S_seq + 31) / 32) * N_heads * S_mb >= 256 ? 2 : 1; }

template <typename T, int VEC, int RT, int DP>
bf_status fwd_rt(int S_mb, int S_seq, int N_heads, int d, int causal, const void* qkv, void* ctx, float* lse, hipStream_t st) {
  const size_t dyn = fwd_scores_bytes(RT, S_seq);
  auto kern = attn_fwd_f32_kernel<T, VEC, RT, DP>;
  if (dyn + fwd_fixed_bytes(RT, DP) > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn);
    if (e != hipSuccess) { set_error("attention_f32: cannot reserve %zu bytes of LDS: %s", dyn, hipGetErrorString(e)); return BF_EDEVICE; }
  }
  kern<<<dim3((S_seq + 16 * RT - 1) / (16 * RT), N_heads, S_mb), NT, dyn, st>>>((const T*)qkv, (T*)ctx, lse, S_seq, N_heads, d, causal,
                                                                               1.0f / sqrtf((float)d));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_error("attention_fwd_f32 launch failed: %s", hipGetErrorString(e)); return BF_EDEVICE; }
  return BF_OK;
}

template <typename T, int VEC, int RT, int DP>
bf_status bwd_rt(int S_mb, int S_seq, int N_heads, int d, int causal, const void* qkv, const float* lse, const float* delta,
                 const void* dctx, void* dqkv, hipStream_t st) {
  const dim3 grid((S_seq + 16 * RT - 1) / (16 * RT), N_heads, S_mb);
  const float scale = 1.0f / sqrtf((float)d);
  attn_bwd_dq_f32_kernel<T, VEC, RT, DP><<<grid, NT, 0, st>>>((const T*)qkv, (const T*)dctx, lse, delta, (T*)dqkv, S_seq, N_heads, d, causal, scale);
  attn_bwd_dkv_f32_kernel<T, VEC, RT, DP><<<grid, NT, 0, st>>>((const T*)qkv, (const T*)dctx, lse, delta, (T*)dqkv, S_seq, N_heads, d, causal, scale);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_error("attention_bwd_f32 launch failed: %s", hipGetErrorString(e)); return BF_EDEVICE; }
  return BF_OK;
}

// calls f(integral constant of VEC, of the padded head size) for a head size that fits
template <typename T, typename F>
bf_status by_head(int d, const void* p0, const void* p1, F f) {
  const bool vec = d % 4 == 0 && (((uintptr_t)p0 | (uintptr_t)p1) & (4 * sizeof(T) - 1)) == 0;
  typedef std::integral_constant<int, 4> V4;
  typedef std::integral_constant<int, 1> V1;
  typedef std::integral_constant<int, 64> D64;
  typedef std::integral_constant<int, 128> D128;
  if (d <= 64) return vec ? f(V4{}, D64{}) : f(V1{}, D64{});
  return vec ? f(V4{}, D128{}) : f(V1{}, D128{});
}

}  // namespace

bool attention_f32_supported(int S_mb, int S_seq, int N_heads, int S_head) {
  return S_mb >= 1 && N_heads >= 1 && S_mb <= 65535 && N_heads <= 65535 && S_seq >= 1 && S_seq <= 4096 && S_head >= 1 && S_head <= 128;
}

// The scores of 16 rows have to fit beside the tiles (S_seq up to 1856 at head sizes up to 128, 2176 up to 64).
bool attention_fwd_f32_supported(int S_mb, int S_seq, int N_heads, int S_head) {
  return attention_f32_supported(S_mb, S_seq, N_heads, S_head) &&
         fwd_scores_bytes(1, S_seq) + fwd_fixed_bytes(1, S_head <= 64 ? 64 : 128) <= LDS_MAX;
}

// Where they are faster than the plain kernels (same bits).  Forward: a tile of 64 keys costs two barriers and products over
// heads padded to 64 or 128, so short rows on a mostly idle chip and small heads stay with the plain kernel.  One idle-chip
// row against the plain kernel's: S_seq 128, one head of 64, fp32 0.96 of its time, 96 1.11; 400, 32 1.04; 64, 96 0.92; with the
// chip full, 64 heads of 32 at S_seq 64 0.83, 16 heads at 128 0.93; bf16 loads are the plain kernel's cheaper ones: 128, one
// head of 96 0.92, 96 1.04.  Heads up to 24: 64 heads of 8 at S_seq 256 0.63, at 400 1.19, at 1000 1.35 (the scores of long rows
// leave room for fewer workgroups); fp32 heads of 24 keep ahead there, 16 heads at 1000 0.77.
// Backward: 48 rows on (S_seq 16, 64 heads of 96 1.2; 48 1.02 at most), with wide or many heads 32 (64 heads of 64 0.7).
bool attention_fwd_f32_better(int dtype, int S_mb, int S_seq, int N_heads, int S_head) {
  const bool b16 = dtype == BF_BF16;
  const long rows = (long)S_mb * S_seq * N_heads, d = S_head;
  if (d <= 16 || (d <= 24 && b16)) return S_seq >= 192 && S_seq <= 256 && rows >= (b16 ? 8192 : 4096);
  if (d <= 24) return S_seq >= 192 && rows >= 3072;
  return S_seq >= 64 && (S_seq * d * d * d >= (b16 ? 100000000 : 1 << 25) || rows >= (b16 ? 4096 : 3072));
}

bool attention_bwd_f32_better(int S_mb, int S_seq, int N_heads, int S_head) {
  return S_seq >= 48 || (S_seq >= 32 && (S_head > 64 || (S_head >= 32 && (long)S_mb * S_seq * N_heads >= 2048)));
}

template <typename T>
static bf_status fwd_f32_t(int S_mb, int S_seq, int N_heads, int d, int causal, const void* qkv, void* ctx, float* lse, hipStream_t st) {
  return by_head<T>(d, qkv, qkv, [&](auto vc, auto dc) {
    constexpr int V = decltype(vc)::value, DP = decltype(dc)::value;
    const bool two = row_tiles(S_mb, S_seq, N_heads) == 2 && fwd_scores_bytes(2, S_seq) + fwd_fixed_bytes(2, DP) <= LDS_MAX;
    return two ? fwd_rt<T, V, 2, DP>(S_mb, S_seq, N_heads, d, causal, qkv, ctx, lse, st)
               : fwd_rt<T, V, 1, DP>(S_mb, S_seq, N_heads, d, causal, qkv, ctx, lse, st);
  });
}

bf_status attention_fwd_f32(int dtype, int S_mb, int S_seq, int N_heads, int S_head, int causal, const void* qkv, void* ctx, float* lse,
                            hipStream_t st) {
  if (!attention_fwd_f32_supported(S_mb, S_seq, N_heads, S_head)) { set_error("attention_fwd_f32: shape not supported"); return BF_EINVAL; }
  return dtype == BF_BF16 ? fwd_f32_t<bf16_t>(S_mb, S_seq, N_heads, S_head, causal, qkv, ctx, lse, st)
                          : fwd_f32_t<float>(S_mb, S_seq, N_heads, S_head, causal, qkv, ctx, lse, st);
}

template <typename T>
static bf_status bwd_f32_t(int S_mb, int S_seq, int N_heads, int d, int causal, const void* qkv, const float* lse, const float* delta,
                           const void* dctx, void* dqkv, hipStream_t st) {
  return by_head<T>(d, qkv, dctx, [&](auto vc, auto dc) {
    constexpr int V = decltype(vc)::value, DP = decltype(dc)::value;
    return row_tiles(S_mb, S_seq, N_heads) == 2 ? bwd_rt<T, V, 2, DP>(S_mb, S_seq, N_heads, d, causal, qkv, lse, delta, dctx, dqkv, st)
                                                : bwd_rt<T, V, 1, DP>(S_mb, S_seq, N_heads, d, causal, qkv, lse, delta, dctx, dqkv, st);
  });
}

// delta[b, head, i] = sum_c dctx ctx has to be there already
bf_status attention_bwd_f32(int dtype, int S_mb, int S_seq, int N_heads, int S_head, int causal, const void* qkv, const float* lse,
                            const float* delta, const void* dctx, void* dqkv, hipStream_t st) {
  if (!attention_f32_supported(S_mb, S_seq, N_heads, S_head)) { set_error("attention_bwd_f32: shape not supported"); return BF_EINVAL; }
  return dtype == BF_BF16 ? bwd_f32_t<bf16_t>(S_mb, S_seq, N_heads, S_head, causal, qkv, lse, delta, dctx, dqkv, st)
                          : bwd_f32_t<float>(S_mb, S_seq, N_heads, S_head, causal, qkv, lse, delta, dctx, dqkv, st);
}

}  // namespace bf
