// What the attention kernels on the bf16 matrix cores share: LDS tiles and their swizzle, fragments, column sums.  The
// accumulator and operand layouts are described in attention_mfma.hip.
#pragma once
#include <float.h>

#include "common.h"

namespace bf {

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

constexpr int NTHR = 256;   // 4 waves; wave w owns rows 32w..32w+31 of the workgroup's 128-row block
constexpr int WG_ROWS = 128;
constexpr int BLK = 64;     // rows of the streamed tiles (keys in forward/dQ, queries in dK/dV)
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

// XOR key of a tile row.  The LDS has 64 banks of 4 bytes; a 16-byte-per-lane read is served 16
// lanes (16 rows, one logical chunk) at a time and a transpose load 32 lanes (4 rows x 4
// adjacent chunks) at a time.  Both sets land in 16 distinct 16-byte slots of the 256-byte bank
// line when the key sends row bits 0-1 to chunk bits 2-3 and row bits 2-3 to chunk bits 0-1
// (S_head 128: 16 chunks per 256-byte row), or row bit 1 to chunk bit 2 and row bits 2-3 to chunk
// bits 0-1 with the row parity choosing the half line (S_head 64: 8 chunks per 128-byte row).
template <int D>
__device__ __forceinline__ int row_key(int row) {
  return D == 128 ? (((row & 3) << 2) | ((row >> 2) & 3)) : ((((row >> 1) & 1) << 2) | ((row >> 2) & 3));
}

template <int D>
__device__ __forceinline__ int swz(int row, int col) {
  return row * D + ((((col >> 3) ^ row_key<D>(row)) << 3) | (col & 7));
}

// thread's 16-byte chunks of a [ROWS][D] tile
template <int ROWS, int D, int NT = 256>
struct TileRegs {
  static constexpr int CH = ROWS * D / 8 / NT;
  u32x4 v[CH];
  __device__ __forceinline__ void load(const bf16_t* __restrict__ g, size_t ld, int tid) {
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int c = tid + i * NT, row = c / (D / 8), ch = c % (D / 8);
      v[i] = *reinterpret_cast<const u32x4*>(g + (size_t)row * ld + ch * 8);
    }
  }
  // rows from `valid` >= 1 on (the sequence ends inside the tile) repeat the last valid one
  __device__ __forceinline__ void load_edge(const bf16_t* __restrict__ g, size_t ld, int tid, int valid) {
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int c = tid + i * NT, row = min(c / (D / 8), valid - 1), ch = c % (D / 8);
      v[i] = *reinterpret_cast<const u32x4*>(g + (size_t)row * ld + ch * 8);
    }
  }
  __device__ __forceinline__ void store(bf16_t* lds, int tid) const {
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int c = tid + i * NT, row = c / (D / 8), ch = c % (D / 8);
      *reinterpret_cast<u32x4*>(lds + row * D + ((ch ^ row_key<D>(row)) << 3)) = v[i];
    }
  }
  // an infinity or a NaN among the thread's values: an exponent of all ones carries into the sign's place
  __device__ __forceinline__ bool non_finite() const {
    uint32_t carry = 0;
#pragma unroll
    for (int i = 0; i < CH; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) carry |= (v[i][j] & 0x7f807f80u) + 0x00800080u;
    return (carry & 0x80008000u) != 0;
  }
};

// A operand, contraction along the tile's columns: lane holds tile[row0 + l%32][16kk + 8(l/32) .. +7]
template <int D>
__device__ __forceinline__ bf16x8 frag_k(const bf16_t* tile, int row0, int kk, int lane) {
  return *reinterpret_cast<const bf16x8*>(tile + swz<D>(row0 + (lane & 31), kk * 16 + 8 * (lane >> 5)));
}

// A operand, contraction along the tile's rows in the accumulator order: lane holds
// tile[rowbase + 8(e/4) + 4(l/32) + e%4][col0 + l%32] for e = 0..7
template <int D>
__device__ __forceinline__ bf16x8 frag_t(const bf16_t* tile, int rowbase, int col0, int lane) {
  const int t = lane & 15, blk = lane >> 4;
  const int row = rowbase + 4 * (blk >> 1) + (t >> 2);
  const int col = col0 + 16 * (blk & 1) + 4 * (t & 3);
  typedef s16x4 __attribute__((address_space(3))) * lds_v4;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(tile + swz<D>(row, col)));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(tile + swz<D>(row + 8, col)));
  return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// registers 8kk..8kk+7 of an accumulator tile as a bf16 B operand
__device__ __forceinline__ bf16x8 pack8(const f32x16& a, int kk) {
  bf16x8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = (__bf16)a[8 * kk + e];
  return o;
}

// two values as a pair of bf16, and what the pair leaves of them (each difference is exact)
__device__ __forceinline__ uint32_t take_bf16(float& a, float& b) {
  typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
  typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
  const uint32_t u = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
  a -= __builtin_bit_cast(float, u << 16);
  b -= __builtin_bit_cast(float, u & 0xffff0000u);
  return u;
}

// the same as three B operands that add up to the 24 bits of the fp32 values.  In pairs, as the conversion instruction takes them:
// value by value the first two parts were converted twice, 7.5 instructions for each in place of 5.5.
__device__ __forceinline__ void pack8_parts(const f32x16& a, int kk, bf16x8& hi, bf16x8& mid, bf16x8& lo) {
  u32x4 part[3];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float v = a[8 * kk + 2 * e], w = a[8 * kk + 2 * e + 1];
#pragma unroll
    for (int q = 0; q < 3; ++q) part[q][e] = take_bf16(v, w);
  }
  hi = __builtin_bit_cast(bf16x8, part[0]);
  mid = __builtin_bit_cast(bf16x8, part[1]);
  lo = __builtin_bit_cast(bf16x8, part[2]);
}

// ---- Sequences of any length (the EDGE forms of the kernels below).  Tiles past the end are filled with copies of the last
// row and masked: no key makes a copy's score a NaN that does not make the real one's a NaN, as a zero row times an
// infinite key would.  These lengths used to run on fp32 kernels, so probabilities and their gradients keep their 24 bits:
// they enter the products as three bf16 operands.  (Two, 16 bits, are 4 % faster at S_head 128 and 10-20 % at 64, but nearly
// uniform rows over values that cancel were 10 to 30 % further from the exact results than those kernels'.)
// 2 x 1000 tokens, 16 heads of 128, causal, forward / backward: 422 / 911 us on fp32 matrix instructions, 45 / 126 here (bound
// by the chain score -> exponential -> three-part product of one or two waves per SIMD); 4 x 1000, 16 heads of 64,
// bidirectional: 51 / 175.
// A zero times an infinity is a NaN in a matrix instruction, but a masked pair must not touch its row, and neither must the
// smaller parts of a probability (zero or negative) take an infinity's sign: where a tile holds non-finite values, or a score
// gradient is past what bf16 holds, the tile's rows are added element by element, allowed pairs only.
// acc (rows = head dims, column = this lane's row) += sum over the tile's rows of s (rows = tile rows) x tile.
constexpr int DUMP = 16 * 32;  // fp32 words of LDS a wave needs for it
template <int D, int NTT, typename F>
__device__ __forceinline__ void accumulate_allowed(f32x16 (&acc)[D / 32], const f32x16 (&s)[NTT], int t0, const bf16_t* tile, float* dump, int lane, F allowed) {
#pragma unroll 1
  for (int q = 0; q < 2 * NTT; ++q) {  // 16 tile rows at a time: registers 8 (q & 1) .. of s[q / 2]
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float v = s[0][e];
#pragma unroll
      for (int u = 1; u < 2 * NTT; ++u) v = u == q ? s[u / 2][8 * (u & 1) + e] : v;
      dump[((e >> 2) * 8 + (lane >> 5) * 4 + (e & 3)) * 32 + (lane & 31)] = v;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll 1
    for (int k = 0; k < 16; ++k) {
      const int row = 32 * t0 + 16 * q + k;
      if (!allowed(row)) continue;
      const float p = dump[k * 32 + (lane & 31)];
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[dt][r] = fmaf(p, (float)tile[swz<D>(row, 32 * dt + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3))], acc[dt][r]);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
}

// a value of the wave's that would round to an infinity (a NaN stays one either way)
template <int NTT>
__device__ __forceinline__ bool past_bf16(const f32x16 (&s)[NTT]) {
  float m = 0.f;
#pragma unroll
  for (int u = 0; u < NTT; ++u)
#pragma unroll
    for (int r = 0; r < 16; ++r) m = fmaxf(m, fabsf(s[u][r]));
  return __builtin_amdgcn_ballot_w64(m > 0x1.fep127f) != 0;
}

// B operand straight from global memory: lane holds row[16kk + 8(l/32) .. +7] of its own token row
template <int D>
__device__ __forceinline__ void load_rowfrags(const bf16_t* __restrict__ row, int lane, bf16x8 (&f)[D / 16]) {
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) f[kk] = *reinterpret_cast<const bf16x8*>(row + kk * 16 + 8 * (lane >> 5));
}

// Scheduling hint for a run of NMMA MFMAs that each consume RPM LDS reads: the reads run AHEAD
// MFMAs in front of their use (an LDS read takes a few MFMA times to return), then nothing moves
// across the end of the run.
template <int NMMA, int RPM, int AHEAD>
__device__ __forceinline__ void mfma_lds_pipeline() {
  __builtin_amdgcn_sched_group_barrier(0x100, AHEAD * RPM, 0);
#pragma unroll
  for (int i = 0; i < NMMA - AHEAD; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, RPM, 0);
  }
  __builtin_amdgcn_sched_group_barrier(0x008, AHEAD, 0);
  __builtin_amdgcn_sched_barrier(0);
}

// acc += tile^T s over the 32 tile rows from row0 on, s (fp32 accumulator layout) in three parts, the smallest first
template <int D, typename FA>
__device__ __forceinline__ void accumulate_split(f32x16 (&acc)[D / 32], const f32x16& s, const bf16_t* tile, int row0, const FA& fa) {
#pragma unroll
  for (int k2 = 0; k2 < 2; ++k2) {
    bf16x8 part[3], tf[D / 32];
    pack8_parts(s, k2, part[2], part[1], part[0]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) tf[dt] = fa.frag_t(tile, row0 + 16 * k2, dt);
    // a part over all head dimensions, then the next: the three products into one accumulator do not wait for each other
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int dt = 0; dt < D / 32; ++dt) acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tf[dt], part[q], acc[dt], 0, 0, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);  // two fragments (two reads each) ahead of the first products
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (dt + 2 < D / 32) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 2 * (D / 32), 0);
    __builtin_amdgcn_sched_barrier(0);
  }
}

__device__ __forceinline__ int acc_row(int r, int lane) { return (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3); }

__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.f;
  return z;
}

// store a transposed accumulator set acc[dt] (rows = head dims, column = this lane's token) as a token row
template <int D>
__device__ __forceinline__ void store_rows(const f32x16 (&acc)[D / 32], bf16_t* __restrict__ row, int lane, float mul) {
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      bf16x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (__bf16)(acc[dt][q4 * 4 + e] * mul);
      *reinterpret_cast<bf16x4*>(row + dt * 32 + q4 * 8 + (lane >> 5) * 4) = o;
    }
}

// ---- column sums of a transposed accumulator set over a workgroup's tokens (the bias gradient of the QKV
// projection is the column sum of dqkv: taking it here saves a second pass over that tensor).
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  const int i = __builtin_bit_cast(int, v);  // every lane has a source under these controls: `old` is never taken
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(i, i, CTRL, 0xf, 0xf, true));
}
// every lane gets the sum over its row of 16 lanes: neighbours in a quad, the other pair of the quad, the
// mirrored half of 8, the mirrored half of 16
__device__ __forceinline__ float row16_sum(float v) {
  v += dpp_f32<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  v += dpp_f32<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v += dpp_f32<0x141>(v);  // row_half_mirror
  v += dpp_f32<0x140>(v);  // row_mirror
  return v;
}
// acc[dt][r] of lane l is head dimension 32 dt + acc_row(r, l) of token l % 32.  The wave leaves the sums over
// each of its four rows of 16 lanes in red[row][16 dt + r] (rows 0-1: lanes 0-31, rows 2-3: lanes 32-63).
template <int D>
__device__ __forceinline__ void wave_colsum(const f32x16 (&acc)[D / 32], float mul, float* red, int lane) {
  f32x16 v[D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) v[dt][r] = row16_sum(acc[dt][r] * mul);
  if ((lane & 15) == 0) {  // one lane per row stores the row's D / 2 sums, 16 bytes at a time
    f32x4* dst = reinterpret_cast<f32x4*>(red + (lane >> 4) * (D / 2));
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        f32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = v[dt][q4 * 4 + e];
        dst[dt * 4 + q4] = o;
      }
  }
}
// head dimension d of the workgroup's column sums: waves w0 .. w0 + nw - 1 of red ([wave][4][D / 2]) in order
template <int D>
__device__ __forceinline__ float colsum_of(const float* red, int w0, int nw, int d) {
  const int dt = d >> 5, rem = d & 31, r = ((rem >> 3) << 2) | (rem & 3), hh = (rem >> 2) & 1;
  float t = 0.f;
  for (int w = w0; w < w0 + nw; ++w) {
    const float* rw = red + (size_t)w * 4 * (D / 2) + dt * 16 + r;
    t += rw[(2 * hh) * (D / 2)] + rw[(2 * hh + 1) * (D / 2)];
  }
  return t;
}

// Per-lane LDS offsets of the fragment reads.  The XOR swizzle makes an address a non-linear
// function of (row, chunk), but the key depends on the lane's row modulo 16 only, so a lane has one
// offset per distinct chunk pattern; tile row blocks of 16 / 32 rows and the LDS stage then enter as
// compile-time constants that the DS instructions take as immediates instead of a shift / xor / add
// chain per read.
template <int D>
struct FragAddr {
  int k[D / 16];      // frag_k, rows 0-31: element offset of chunk 2kk + lane/32 of row lane%32
  int t[2][D / 32];   // frag_t, row block 0: offsets of the two transpose loads (rows r, r+8) per 32-column block
  __device__ __forceinline__ void init(int lane) {
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) k[kk] = swz<D>(lane & 31, kk * 16 + 8 * (lane >> 5));
    const int tt = lane & 15, blk = lane >> 4;
    const int row = 4 * (blk >> 1) + (tt >> 2), col = 16 * (blk & 1) + 4 * (tt & 3);
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) {
      t[0][dt] = swz<D>(row, 32 * dt + col);
      t[1][dt] = swz<D>(row + 8, 32 * dt + col);
    }
  }
  // A operand, contraction along the tile's columns: lane holds tile[row0 + l%32][16kk + 8(l/32) .. +7]; row0 % 16 == 0
  __device__ __forceinline__ bf16x8 frag_k(const bf16_t* tile, int row0, int kk) const {
    return *reinterpret_cast<const bf16x8*>(tile + row0 * D + k[kk]);
  }
  // A operand, contraction along the tile's rows in the accumulator order: lane holds
  // tile[rowbase + 8(e/4) + 4(l/32) + e%4][32 dt + l%32] for e = 0..7; rowbase % 16 == 0
  __device__ __forceinline__ bf16x8 frag_t(const bf16_t* tile, int rowbase, int dt) const {
    typedef s16x4 __attribute__((address_space(3))) * lds_v4;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(tile + rowbase * D + t[0][dt]));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(tile + rowbase * D + t[1][dt]));
    return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }
};

// The same interface from two registers: chunk and key occupy different bits, so every offset is the first one of its kind XOR a
// constant (eight rows on flips bit 1 of the key), one instruction with the addition of the tile's address.  `loop` at the
// head of a loop keeps the compiler from computing them all in front of it, into the registers that this form is to save.
template <int D>
struct FragAddrXor {
  int k0, t0;
  __device__ __forceinline__ void init(int lane) {
    const int tt = lane & 15, blk = lane >> 4;
    k0 = swz<D>(lane & 31, 8 * (lane >> 5));
    t0 = swz<D>(4 * (blk >> 1) + (tt >> 2), 16 * (blk & 1) + 4 * (tt & 3));
  }
  __device__ __forceinline__ void loop() { asm volatile("" : "+v"(k0), "+v"(t0)); }
  __device__ __forceinline__ bf16x8 frag_k(const bf16_t* tile, int row0, int kk) const {
    return *reinterpret_cast<const bf16x8*>(tile + row0 * D + (k0 ^ (16 * kk)));
  }
  __device__ __forceinline__ bf16x8 frag_t(const bf16_t* tile, int rowbase, int dt) const {
    typedef s16x4 __attribute__((address_space(3))) * lds_v4;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(tile + rowbase * D + (t0 ^ (32 * dt))));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)(tile + (rowbase + 8) * D + (t0 ^ (32 * dt) ^ 16)));
    return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }
};

// The same interface computing every address on the fly: for kernels that have no 16 registers to spare.
template <int D>
struct FragAddrLive {
  int lane_;
  __device__ __forceinline__ void init(int lane) { lane_ = lane; }
  __device__ __forceinline__ bf16x8 frag_k(const bf16_t* tile, int row0, int kk) const { return bf::frag_k<D>(tile, row0, kk, lane_); }
  __device__ __forceinline__ bf16x8 frag_t(const bf16_t* tile, int rowbase, int dt) const { return bf::frag_t<D>(tile, rowbase, 32 * dt, lane_); }
};

}  // namespace
}  // namespace bf
