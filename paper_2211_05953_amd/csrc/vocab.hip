// Input and output layers of the language model (App. A.1; the S_voc term of Eq. compute):
// token + position embedding forward and backward, softmax cross-entropy with its gradient
// written in place of the logits.  The projections themselves are the GEMM kernels.
// All HBM-bound row kernels: one 256-thread workgroup per token row.  Every sum has a fixed
// order (no atomics), so the gradients do not depend on scheduling.
#include <math.h>

#include "common.h"

namespace bf {

namespace {

constexpr int ROW_THREADS = 256;

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

inline bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

template <typename T, int VEC>
struct alignas(sizeof(T) * VEC > 16 ? 16 : sizeof(T) * VEC) Vec {
  T v[VEC];
};

template <typename T, int VEC>
__device__ __forceinline__ void load_vec(const T* p, float (&out)[VEC]) {
  typedef Vec<T, VEC> V;
  V t = *reinterpret_cast<const V*>(p);
#pragma unroll
  for (int i = 0; i < VEC; ++i) out[i] = (float)t.v[i];
}

template <typename T, int VEC>
__device__ __forceinline__ void store_vec(T* p, const float (&in)[VEC]) {
  typedef Vec<T, VEC> V;
  V t;
#pragma unroll
  for (int i = 0; i < VEC; ++i) t.v[i] = (T)in[i];
  *reinterpret_cast<V*>(p) = t;
}

// x[t, :] = E_tok[tok[t], :] + E_pos[t mod S_seq, :]; an id outside 0..S_voc-1 contributes no token row.
template <typename T, int VEC>
__global__ __launch_bounds__(ROW_THREADS) void embedding_fwd_kernel(const int32_t* __restrict__ tok,
                                                                    const float* __restrict__ e_tok,
                                                                    const float* __restrict__ e_pos, T* __restrict__ x,
                                                                    int S_seq, int S_voc, int h) {
  const size_t row = blockIdx.x;
  const int v = tok[row];
  const bool valid = v >= 0 && v < S_voc;
  const float* er = e_tok + (size_t)(valid ? v : 0) * h;
  const float* pr = e_pos + (row % (size_t)S_seq) * h;
  T* xr = x + row * (size_t)h;
  for (int c = threadIdx.x * VEC; c < h; c += ROW_THREADS * VEC) {
    float a[VEC], b[VEC];
    load_vec<float, VEC>(er + c, a);
    load_vec<float, VEC>(pr + c, b);
#pragma unroll
    for (int j = 0; j < VEC; ++j) a[j] = (valid ? a[j] : 0.f) + b[j];
    store_vec<T, VEC>(xr + c, a);
  }
}

// How many of the workgroup's threads say yes, in one barrier; `slot` must not be written again before all have read it.
__device__ __forceinline__ int count_threads(bool yes, int (&slot)[ROW_THREADS / 64]) {
  const int n = __popcll(__ballot(yes));
  if ((threadIdx.x & 63) == 0) slot[threadIdx.x >> 6] = n;
  __syncthreads();
  int sum = 0;
#pragma unroll
  for (int q = 0; q < ROW_THREADS / 64; ++q) sum += slot[q];
  return sum;
}

// Token- and position-embedding gradients in one launch, without atomics.  Workgroups x < n_rows: the one of the first
// position that uses a token sums the rows of every position using it, in ascending position, and adds the sum to that
// token's gradient row; workgroups of later uses leave at once.  Distinct tokens, distinct rows.  The others: position
// i sums its row over the samples of the micro-batch.
// Two things bound the launch.  A frequent token's workgroup is the longest (300 of 2048 positions under a Zipf law), by the
// latency and the bytes of its rows: UN of them are in flight at a time (added in their order), and its columns are split
// over the workgroups of grid.y.  And every workgroup of a first position reads all the ids, which with few repeats is
// n^2 reads: there only workgroup y = 0 does, and sums all the columns.  A token is frequent where FN pairs of
// positions 256 apart in the FW from t on use it (one barrier); which side a token falls on changes no bit of its sum.
// One row at a time and one wavefront searching / the columns of all tokens split / this, bf16, 50304 ids, us: 2048 tokens of 2048
// columns, frequent ones among them 208 / 27 / 27, uniform 18 / 23 / 18; 16384 of 4096 4039 / 699 / 322 and 420 / 1071 / 298.
template <typename T, int VEC>
__global__ __launch_bounds__(ROW_THREADS) void embedding_bwd_kernel(const int32_t* __restrict__ tok, const T* __restrict__ d,
                                                                    float* __restrict__ g_tok, float* __restrict__ g_pos, int S_mb,
                                                                    int S_seq, int S_voc, int h, int accumulate_pos, int tok16) {
  constexpr int PER = 8, WIN = ROW_THREADS * PER, UN = 16, FW = 2 * ROW_THREADS, FN = 8, CHUNK = ROW_THREADS * VEC;
  typedef Vec<T, VEC> V;
  typedef Vec<int32_t, 4> I4;  // used where tok16: the ids are 16-byte aligned
  const int n_rows = S_mb * S_seq, tid = threadIdx.x;
  if ((int)blockIdx.x >= n_rows) {
    const int i = blockIdx.x - n_rows, c = blockIdx.y * CHUNK + tid * VEC;
    if (c >= h) return;
    float* gr = g_pos + (size_t)i * h + c;
    float acc[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) acc[j] = 0.f;
    for (int b = 0; b < S_mb; ++b) {
      float r[VEC];
      load_vec<T, VEC>(d + ((size_t)b * S_seq + i) * h + c, r);
#pragma unroll
      for (int j = 0; j < VEC; ++j) acc[j] += r[j];
    }
    if (accumulate_pos) {
      float g[VEC];
      load_vec<float, VEC>(gr, g);
#pragma unroll
      for (int j = 0; j < VEC; ++j) acc[j] += g[j];
    }
    store_vec<float, VEC>(gr, acc);
    return;
  }
  __shared__ int list[WIN];
  __shared__ int wave_n[ROW_THREADS / 64], votes[3][ROW_THREADS / 64], hit_votes[2][ROW_THREADS / 64];
  const int t = blockIdx.x;
  const int v = tok[t];
  if (v < 0 || v >= S_voc) return;
  int first_chunk = 0, chunks = gridDim.y;  // of the columns, this workgroup's
  if (n_rows <= FW / 2) {  // reading the ids is nothing
    first_chunk = blockIdx.y;
    chunks = 1;
  } else if (chunks > 1) {
    const int i = t + tid;  // (pairs of positions are counted: one barrier)
    const bool u0 = i < n_rows && tok[i] == v, u1 = i + ROW_THREADS < n_rows && tok[i + ROW_THREADS] == v;
    if (count_threads(u0 || u1, votes[0]) >= FN) {
      first_chunk = blockIdx.y;
      chunks = 1;
    } else if (blockIdx.y) {
      return;
    }
  }
  // an earlier use, among the first positions (a frequent token's is there), then among the others
  int earlier = 0;
  const int near = min(t, 4 * ROW_THREADS);
#pragma unroll 4
  for (int i = tid; i < near; i += ROW_THREADS) earlier |= tok[i] == v;
  if (count_threads(earlier, votes[1])) return;
  if (t > near) {
    if (tok16) {
#pragma unroll 4
      for (int i = near + tid * 4; i + 4 <= t; i += ROW_THREADS * 4) {
        const I4 u = *reinterpret_cast<const I4*>(tok + i);
#pragma unroll
        for (int e = 0; e < 4; ++e) earlier |= u.v[e] == v;
      }
      if (tid < (t & 3)) earlier |= tok[(t & ~3) + tid] == v;
    } else {
#pragma unroll 8
      for (int i = near + tid; i < t; i += ROW_THREADS) earlier |= tok[i] == v;
    }
    if (count_threads(earlier, votes[2])) return;
  }
  const int lane = tid & 63, w = tid >> 6;
  // The positions that use the token, a window at a time (one without it costs a barrier).  Windows share the list while it
  // has room; a chunk of columns is summed from it in one go, or, where the uses did not fit, list after list.
  int w0 = 0, n = 0, turn = 0;  // the next window, entries of the list, which votes
  bool whole = true;  // the list has held all uses since the first window
  auto fill = [&] {   // false: no more windows, or no room for this one's uses
    if (w0 >= n_rows) return false;
    const int i0 = w0 + tid * PER;
    unsigned hits = 0;
    if (tok16 && i0 + PER <= n_rows) {
#pragma unroll
      for (int q = 0; q < PER / 4; ++q) {
        const I4 u = *reinterpret_cast<const I4*>(tok + i0 + 4 * q);
#pragma unroll
        for (int e = 0; e < 4; ++e) hits |= (u.v[e] == v ? 1u : 0u) << (4 * q + e);
      }
    } else {
#pragma unroll
      for (int e = 0; e < PER; ++e)
        if (i0 + e < n_rows && tok[i0 + e] == v) hits |= 1u << e;
    }
    turn ^= 1;
    if (!count_threads(hits != 0, hit_votes[turn])) {  // (also: wave_n and the votes before have been read)
      w0 += WIN;
      return true;
    }
    int before = __popc(hits);  // hits of the wave's lanes up to this one
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int x = __shfl_up(before, o, 64);
      if (lane >= o) before += x;
    }
    if (lane == 63) wave_n[w] = before;
    before -= __popc(hits);
    __syncthreads();
    int more = 0;
#pragma unroll
    for (int q = 0; q < ROW_THREADS / 64; ++q) {
      if (q < w) before += wave_n[q];
      more += wave_n[q];
    }
    if (n + more > WIN) return false;
    before += n;
#pragma unroll
    for (int e = 0; e < PER; ++e)
      if (hits >> e & 1) list[before++] = i0 + e;
    n += more;
    w0 += WIN;
    return true;
  };
  for (int ch = first_chunk; ch < first_chunk + chunks; ++ch) {
    const int c = ch * CHUNK + tid * VEC;
    float acc[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) acc[j] = 0.f;
    bool last = whole && ch > first_chunk;  // the list is there from the chunk before
    if (!last) w0 = t & ~(PER - 1);         // (positions before t do not use the token)
    for (bool first = true;; first = false) {
      if (!last) {
        if (!first || ch > first_chunk) __syncthreads();  // the list has been read
        n = 0;
        while (fill()) {}
        last = w0 >= n_rows;
        if (!(first && last)) whole = false;
        __syncthreads();
      }
      if (c < h) {
        int k = 0;
        for (; k + UN <= n; k += UN) {
          V r[UN];
#pragma unroll
          for (int u = 0; u < UN; ++u) r[u] = *reinterpret_cast<const V*>(d + (size_t)list[k + u] * h + c);
#pragma unroll
          for (int u = 0; u < UN; ++u)
#pragma unroll
            for (int j = 0; j < VEC; ++j) acc[j] += (float)r[u].v[j];
        }
        for (; k < n; ++k) {
          float r[VEC];
          load_vec<T, VEC>(d + (size_t)list[k] * h + c, r);
#pragma unroll
          for (int j = 0; j < VEC; ++j) acc[j] += r[j];
        }
      }
      if (last) break;
    }
    if (c < h) {
      float* gr = g_tok + (size_t)v * h + c;
      float g[VEC];
      load_vec<float, VEC>(gr, g);
#pragma unroll
      for (int j = 0; j < VEC; ++j) g[j] += acc[j];
      store_vec<float, VEC>(gr, g);
    }
  }
}

// Row-wise softmax cross-entropy.  One pass finds the running maximum and the sum of exponentials
// (rescaled when the maximum moves), a second writes dz = (softmax(z) - onehot(label)) * scale over
// z.  row_loss = (logsumexp(z) - z[label]) * scale.  A label outside 0..S_voc-1 gives a zero row.
template <typename T, int VEC>
__global__ __launch_bounds__(ROW_THREADS) void ce_loss_kernel(T* __restrict__ z, const int32_t* __restrict__ labels,
                                                              float* __restrict__ row_loss, int S_voc, float scale) {
  __shared__ float red_m[4], red_s[4];
  const size_t row = blockIdx.x;
  T* zr = z + row * (size_t)S_voc;
  const int label = labels[row];
  const bool valid = label >= 0 && label < S_voc;
  const float z_label = valid ? (float)zr[label] : 0.f;
  float m = -INFINITY, s = 0.f;
  for (int c = threadIdx.x * VEC; c < S_voc; c += ROW_THREADS * VEC) {
    float v[VEC];
    load_vec<T, VEC>(zr + c, v);
    float cm = v[0];
#pragma unroll
    for (int j = 1; j < VEC; ++j) cm = fmaxf(cm, v[j]);
    if (cm > m) {
      s *= expf(m - cm);  // first chunk: s = 0 and exp(-inf) = 0
      m = cm;
    }
#pragma unroll
    for (int j = 0; j < VEC; ++j) s += expf(v[j] - m);
  }
  // combine the threads: common maximum, sums rescaled to it
  const float wm = wave_max(m);
  s = wave_sum(m == -INFINITY ? 0.f : s * expf(m - wm));  // a thread past the row's end saw nothing
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { red_m[w] = wm; red_s[w] = s; }
  __syncthreads();  // also orders the read of z[label] above before the writes below
  const float M = fmaxf(fmaxf(red_m[0], red_m[1]), fmaxf(red_m[2], red_m[3]));
  float S = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) S += red_m[i] == -INFINITY ? 0.f : red_s[i] * expf(red_m[i] - M);
  const float lse = M + logf(S);
  if (threadIdx.x == 0) row_loss[row] = valid ? (lse - z_label) * scale : 0.f;
  const float sc = valid ? scale : 0.f;
  for (int c = threadIdx.x * VEC; c < S_voc; c += ROW_THREADS * VEC) {
    float v[VEC];
    load_vec<T, VEC>(zr + c, v);
#pragma unroll
    for (int j = 0; j < VEC; ++j) v[j] = (expf(v[j] - lse) - (c + j == label ? 1.f : 0.f)) * sc;
    store_vec<T, VEC>(zr + c, v);
  }
}

// The same with the row in registers between the two passes (NIT vectors of VEC values per thread): the logits are read
// once, and an element's exponential is taken once, for the sum and for its gradient.
// 2048 rows of 50304 in bf16: 154 us (two reads, two exponentials) -> 129 us.
template <typename T, int VEC, int NIT, int NTHR>
__global__ __launch_bounds__(NTHR) void ce_loss_reg_kernel(T* __restrict__ z, const int32_t* __restrict__ labels,
                                                           float* __restrict__ row_loss, int S_voc, float scale) {
  constexpr int NW = NTHR / 64;
  typedef Vec<T, VEC> V;
  __shared__ float red_m[NW], red_s[NW], z_label_s;
  const size_t row = blockIdx.x;
  T* zr = z + row * (size_t)S_voc;
  const int label = labels[row], tid = threadIdx.x, w = tid >> 6;
  const bool valid = label >= 0 && label < S_voc;
  V v[NIT];
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int c = (it * NTHR + tid) * VEC;
    if (c < S_voc) v[it] = *reinterpret_cast<const V*>(zr + c);
  }
  if (tid == 0) z_label_s = valid ? (float)zr[label] : 0.f;  // overwritten only after the barriers below
  float m = -INFINITY;
#pragma unroll
  for (int it = 0; it < NIT; ++it)
    if ((it * NTHR + tid) * VEC < S_voc)
#pragma unroll
      for (int j = 0; j < VEC; ++j) m = fmaxf(m, (float)v[it].v[j]);
  m = wave_max(m);
  if ((tid & 63) == 0) red_m[w] = m;
  __syncthreads();
  float M = red_m[0];
#pragma unroll
  for (int i = 1; i < NW; ++i) M = fmaxf(M, red_m[i]);
  float e[NIT][VEC], s = 0.f;
#pragma unroll
  for (int it = 0; it < NIT; ++it)
    if ((it * NTHR + tid) * VEC < S_voc)
#pragma unroll
      for (int j = 0; j < VEC; ++j) {
        e[it][j] = expf((float)v[it].v[j] - M);
        s += e[it][j];
      }
  s = wave_sum(s);
  if ((tid & 63) == 0) red_s[w] = s;
  __syncthreads();
  float S = 0.f;
#pragma unroll
  for (int i = 0; i < NW; ++i) S += red_s[i];
  if (tid == 0) row_loss[row] = valid ? (M + logf(S) - z_label_s) * scale : 0.f;
  const float sc = valid ? scale : 0.f, inv = 1.0f / S;
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int c = (it * NTHR + tid) * VEC;
    if (c < S_voc) {
#pragma unroll
      for (int j = 0; j < VEC; ++j) e[it][j] = (e[it][j] * inv - (c + j == label ? 1.f : 0.f)) * sc;
      store_vec<T, VEC>(zr + c, e[it]);
    }
  }
}

// Rows of whole 16-byte vectors that fit the registers of 256, 512 or 1024 threads; false: the two-pass kernel's.  (1024
// threads with a quarter of their places taken lose to that: 8192 rows of 8200 in bf16 82 us there, 111 on 1024, 59 on 512.)
template <typename T, int VEC>
bool launch_ce_reg(int n_rows, int S_voc, void* z, const int32_t* labels, float scale, float* row_loss, hipStream_t st) {
  if (S_voc % VEC || ((uintptr_t)z & 15)) return false;
  const int nv = S_voc / VEC;
  if (nv <= 256) ce_loss_reg_kernel<T, VEC, 1, 256><<<n_rows, 256, 0, st>>>((T*)z, labels, row_loss, S_voc, scale);
  else if (nv <= 1024) ce_loss_reg_kernel<T, VEC, 4, 256><<<n_rows, 256, 0, st>>>((T*)z, labels, row_loss, S_voc, scale);
  else if (nv <= 2 * 1024) ce_loss_reg_kernel<T, VEC, 4, 512><<<n_rows, 512, 0, st>>>((T*)z, labels, row_loss, S_voc, scale);
  else if (nv <= 4 * 1024) ce_loss_reg_kernel<T, VEC, 4, 1024><<<n_rows, 1024, 0, st>>>((T*)z, labels, row_loss, S_voc, scale);
  else if (nv <= 7 * 1024) ce_loss_reg_kernel<T, VEC, 7, 1024><<<n_rows, 1024, 0, st>>>((T*)z, labels, row_loss, S_voc, scale);
  else if (VEC == 4 && nv <= 13 * 1024) ce_loss_reg_kernel<T, VEC, VEC == 4 ? 13 : 1, 1024><<<n_rows, 1024, 0, st>>>((T*)z, labels, row_loss, S_voc, scale);
  else return false;
  return true;
}

// out[0] = sum of n values, fixed order: strided partial sums per thread, then a tree.
__global__ __launch_bounds__(ROW_THREADS) void sum_rows_kernel(const float* __restrict__ v, float* __restrict__ out, int n) {
  __shared__ float red[ROW_THREADS];
  float s = 0.f;
  for (int i = threadIdx.x; i < n; i += ROW_THREADS) s += v[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = ROW_THREADS / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = red[0];
}


#define BF_LAUNCH_CHECK()                                                                  \
  do {                                                                                     \
    hipError_t e_ = hipGetLastError();                                                     \
    if (e_ != hipSuccess) { set_error("kernel launch failed: %s", hipGetErrorString(e_)); return BF_EDEVICE; } \
  } while (0)

}  // namespace

bf_status embedding_fwd(int dtype, int n_rows, int S_seq, int S_voc, int h, const int32_t* tok, const float* e_tok,
                        const float* e_pos, void* x, hipStream_t st) {
  if (n_rows < 1 || S_seq < 1 || S_voc < 1 || h < 1 || !tok || !e_tok || !e_pos || !x) { set_error("embedding_fwd: bad argument"); return BF_EINVAL; }
  const bool vec = h % 4 == 0 && aligned16(e_tok) && aligned16(e_pos) && aligned16(x);
  if (dtype == BF_BF16) {
    if (vec) embedding_fwd_kernel<bf16_t, 4><<<n_rows, ROW_THREADS, 0, st>>>(tok, e_tok, e_pos, (bf16_t*)x, S_seq, S_voc, h);
    else embedding_fwd_kernel<bf16_t, 1><<<n_rows, ROW_THREADS, 0, st>>>(tok, e_tok, e_pos, (bf16_t*)x, S_seq, S_voc, h);
  } else {
    if (vec) embedding_fwd_kernel<float, 4><<<n_rows, ROW_THREADS, 0, st>>>(tok, e_tok, e_pos, (float*)x, S_seq, S_voc, h);
    else embedding_fwd_kernel<float, 1><<<n_rows, ROW_THREADS, 0, st>>>(tok, e_tok, e_pos, (float*)x, S_seq, S_voc, h);
  }
  BF_LAUNCH_CHECK();
  return BF_OK;
}

bf_status embedding_bwd(int dtype, int S_mb, int S_seq, int S_voc, int h, const int32_t* tok, const void* d, float* g_tok,
                        float* g_pos, int accumulate_pos, hipStream_t st) {
  if (S_mb < 1 || S_seq < 1 || S_voc < 1 || h < 1 || !tok || !d || !g_tok || !g_pos) { set_error("embedding_bwd: bad argument"); return BF_EINVAL; }
  const bool vec = h % 4 == 0 && aligned16(d) && aligned16(g_tok) && aligned16(g_pos);
  const int per = ROW_THREADS * (vec ? 4 : 1), tok16 = aligned16(tok) ? 1 : 0;
  const dim3 grid((unsigned)(S_mb * S_seq + S_seq), (unsigned)((h + per - 1) / per));
#define BF_EMB_BWD(T, VEC) \
  embedding_bwd_kernel<T, VEC><<<grid, ROW_THREADS, 0, st>>>(tok, (const T*)d, g_tok, g_pos, S_mb, S_seq, S_voc, h, accumulate_pos, tok16)
  if (dtype == BF_BF16) {
    if (vec) BF_EMB_BWD(bf16_t, 4);
    else BF_EMB_BWD(bf16_t, 1);
  } else {
    if (vec) BF_EMB_BWD(float, 4);
    else BF_EMB_BWD(float, 1);
  }
#undef BF_EMB_BWD
  BF_LAUNCH_CHECK();
  return BF_OK;
}

bf_status ce_loss(int dtype, int n_rows, int S_voc, void* z, const int32_t* labels, float scale, float* row_loss,
                  float* loss_out, hipStream_t st) {
  if (n_rows < 1 || S_voc < 1 || !z || !labels || !row_loss || !loss_out) { set_error("ce_loss: bad argument"); return BF_EINVAL; }
  const bool vec = S_voc % 4 == 0 && aligned16(z);
  if (dtype == BF_BF16 ? launch_ce_reg<bf16_t, 8>(n_rows, S_voc, z, labels, scale, row_loss, st)
                       : launch_ce_reg<float, 4>(n_rows, S_voc, z, labels, scale, row_loss, st)) {
  } else if (dtype == BF_BF16) {
    if (vec) ce_loss_kernel<bf16_t, 4><<<n_rows, ROW_THREADS, 0, st>>>((bf16_t*)z, labels, row_loss, S_voc, scale);
    else ce_loss_kernel<bf16_t, 1><<<n_rows, ROW_THREADS, 0, st>>>((bf16_t*)z, labels, row_loss, S_voc, scale);
  } else {
    if (vec) ce_loss_kernel<float, 4><<<n_rows, ROW_THREADS, 0, st>>>((float*)z, labels, row_loss, S_voc, scale);
    else ce_loss_kernel<float, 1><<<n_rows, ROW_THREADS, 0, st>>>((float*)z, labels, row_loss, S_voc, scale);
  }
  BF_LAUNCH_CHECK();
  sum_rows_kernel<<<1, ROW_THREADS, 0, st>>>(row_loss, loss_out, n_rows);
  BF_LAUNCH_CHECK();
  return BF_OK;
}

}  // namespace bf
