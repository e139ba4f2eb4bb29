// Attention backward for launches that fill the chip: 64 rows per wave instead of 32, so that every 1 KB fragment that is
// read from LDS feeds two matrix products (attention_mfma.hip reads one per product, and that is what bounds its kernels).
// The accumulators and operands of 64 rows at S_head 128 take all 512 registers of a lane, which leaves one wave per SIMD.
// A lone wave issues in order, so whatever it waits for stops its products too; the order of a tile's work is therefore
// fixed by hand, with a scheduling fence per step.  A step is one fragment, the products it feeds and a share of the vector
// work of an earlier phase; fragments are read AHEAD steps before their use and the next tile is requested, and stored to
// the idle LDS stage, a chunk per step.  Layouts, swizzle and the order of sums are those of attention_mfma.hip.
#include <algorithm>
#include <cmath>
#include <type_traits>
#include <utility>

#include "attention_tiles.h"
#include "common.h"

namespace bf {

namespace {

template <typename F, int... I>
__device__ __forceinline__ void static_for_(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) { static_for_(f, std::make_integer_sequence<int, N>{}); }

// f(row) for the share of rows R0 .. R1 - 1 that step C of N takes
template <int R0, int R1, int C, int N, typename F>
__device__ __forceinline__ void share(F&& f) {
  constexpr int r0 = R0 + (R1 - R0) * C / N, r1 = R0 + (R1 - R0) * (C + 1) / N;
  static_for<r1 - r0>([&](auto rc) { f(std::integral_constant<int, r0 + decltype(rc)::value>{}); });
}

typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
__device__ __forceinline__ uint32_t pack2(float a, float b) {
  uint32_t two = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)a, (__bf16)b});
  asm("" : "+v"(two));  // one conversion for both: the halves are unpacked from here, not converted one by one
  return two;
}

// The products, in assembly where 64 rows fill the registers: left to itself the compiler wants every accumulator of the kernel
// in one half of the register file, and they are more than a half.  mfma_v keeps scores where the vector unit reads them,
// mfma_a the sums over tiles in the other half (ASM false: the builtin).  What the compiler then does not see: a product
// must have two issue slots between it and vector instructions that write its operands (`nop` keeps them apart: for the first
// products on new operands, and everywhere outside the loops over tiles, where the compiler may move registers about),
// and there must be 12 between a score's last product and its use (two further products, 16 slots, lie between).  A third operand
// in registers of its own would be read over a product's first 8 slots, and nothing might write those registers for 7 of them;
// there is none here: a sum is its own, and a first product starts from the constant.  tests/test_host_logic.py
// looks for all three in the listing.  Loads into the operands are waited for as usual.
template <bool ASM>
__device__ __forceinline__ void mfma_v(f32x16& c, const bf16x8& a, const bf16x8& b, bool first, bool nop) {
  if constexpr (!ASM) c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, first ? zero16() : c, 0, 0, 0);
  else if (first) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "v"(b));
  else if (nop) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
  else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}
template <bool ASM>
__device__ __forceinline__ void mfma_a(f32x16& c, const bf16x8& a, const bf16x8& b, bool nop) {
  if constexpr (!ASM) c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  else if (nop) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
  else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}
template <bool ASM>
__device__ __forceinline__ void zero_acc(f32x16& c) {
  c = zero16();
  if constexpr (ASM) asm volatile("" : "+a"(c));  // here, not in front of the first product
}
// after the last product, before the sums are read
__device__ __forceinline__ void drain() { asm volatile("s_nop 15\n\ts_nop 7"); }

// Fragment addresses (as FragAddr) formed by an XOR per read, from three registers: the chunk of a read and the key of
// its row meet in disjoint or XORed bits only, and tile row blocks of 16 do not change the key.
template <int D>
struct FragAddrX {
  // (volatile: the compiler would otherwise keep every XORed offset of the loop in a register)
  static __device__ __forceinline__ int flipped(int v, int x) {
    if (x == 0) return v;
    int r;
    asm volatile("v_xor_b32 %0, %1, %2" : "=v"(r) : "i"(x), "v"(v));
    return r;
  }
  int k0, t0, t1;  // bytes: frag_k, chunk 0; frag_t, column block 0, rows r and r + 8
  __device__ __forceinline__ void init(int lane) {
    k0 = 2 * swz<D>(lane & 31, 8 * (lane >> 5));
    const int tt = lane & 15, blk = lane >> 4;
    const int row = 4 * (blk >> 1) + (tt >> 2), col = 16 * (blk & 1) + 4 * (tt & 3);
    t0 = 2 * swz<D>(row, col);
    t1 = 2 * swz<D>(row + 8, col);
  }
  // to the other of two LDS stages that lie `bytes`, a power of two above every offset in a stage, apart
  __device__ __forceinline__ void flip(int bytes) { k0 ^= bytes; t0 ^= bytes; t1 ^= bytes; }
  __device__ __forceinline__ bf16x8 frag_k(const bf16_t* tile, int row0, int kk) const {
    return *reinterpret_cast<const bf16x8*>((const char*)(tile + row0 * D) + flipped(k0, kk * 32));
  }
  __device__ __forceinline__ bf16x8 frag_t(const bf16_t* tile, int rowbase, int dt) const {
    typedef s16x4 __attribute__((address_space(3))) * lds_v4;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)((const char*)(tile + rowbase * D) + flipped(t0, 64 * dt)));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4)((const char*)(tile + rowbase * D) + flipped(t1, 64 * dt)));
    return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }
};

// Two operands' tiles of BLK rows, moved by 256 threads in CH chunks of 16 bytes each, SC of which are in registers at a time.
template <int D, int SC_>
struct TileMover {
  static constexpr int CH = BLK * D / 8 / 256, SC = SC_, NB = 2 * CH / SC, RSTEP = 256 / (D / 8);
  static_assert(RSTEP % 16 == 0, "the swizzle key repeats every 16 rows");
  const bf16_t *src0, *src1;
  int ld0, ld1, off0, off1, lds_off;
  u32x4 stage[SC];
  __device__ __forceinline__ void init(const bf16_t* s0, int l0, const bf16_t* s1, int l1, int tid) {
    src0 = s0; ld0 = l0; src1 = s1; ld1 = l1;
    const int row = tid / (D / 8), ch = tid % (D / 8);
    off0 = (row * ld0 + ch * 8) * 2;
    off1 = (row * ld1 + ch * 8) * 2;
    lds_off = row * D + ((ch ^ row_key<D>(row)) << 3);
  }
  // chunk c of tile j, first operand 0's, then operand 1's; the tile's first row is the buffer's base
  __device__ __forceinline__ void load(int j, int c) {
    const int o = c / CH, i = c % CH;
    const bf16_t* g = o ? src1 + (size_t)j * BLK * ld1 : src0 + (size_t)j * BLK * ld0;
    __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)g, 0, 0x7fffffff, 0x00020000);
    stage[c % SC] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, o ? off1 : off0, i * RSTEP * 2 * (o ? ld1 : ld0), 0);
  }
  __device__ __forceinline__ void store(bf16_t* t, int c) const {
    *reinterpret_cast<u32x4*>(t + (c / CH) * BLK * D + lds_off + (c % CH) * RSTEP * D) = stage[c % SC];
  }
  __device__ __forceinline__ void whole(int j, bf16_t* t) {
#pragma unroll
    for (int n = 0; n < NB; ++n) {
#pragma unroll
      for (int i = 0; i < SC; ++i) load(j, n * SC + i);
#pragma unroll
      for (int i = 0; i < SC; ++i) store(t, n * SC + i);
    }
  }
  // its share of step i of N
  template <int I, int N>
  __device__ __forceinline__ void step(int j, bf16_t* t) {
    constexpr int SHARE = N / NB;
    if constexpr (I % SHARE < SC) load(j, I / SHARE * SC + I % SHARE);
    if constexpr (I % SHARE >= SHARE - SC) store(t, I / SHARE * SC + I % SHARE - (SHARE - SC));
  }
};

// ----------------------------------------------------------------- backward, dK/dV pass
// 4 waves of 32 G keys, each with both gradients of its keys: S and dP, then P and dS from them, all in the wave (the 8-wave
// form hands P from one wave to another).  Every value is rounded where the 128-key form rounds it and every sum has its order, column
// sums included, so the results are the same bits whichever form a launch takes, that is, however many sequences share it.
// (S and dP started from the rows' -lse sqrt(d) and -delta save an operation per element, 1 % of the backward at S_head 128 and 3 %
// at 64, and are other bits.)  Phases of a sub-tile of 32 queries and what runs beside them: S; dP, exponentials of the
// first 10 rows of a lane; dV, the others and dS; dK, the rest of dS.
// Backward of S_head 128, G = 2, S_seq 2048, 64 heads: causal 302 -> 272 us, bidirectional 512 -> 444.  Bound by the products: with
// neither LDS reads, vector work nor the next tile's loads in the loop (bidirectional) 80 % of the kernel's time remains, a
// tenth of it the loads of K and V and the stores at either end, which one workgroup per compute unit cannot hide; without
// the LDS reads 87 %, the vector work 90 %, the loads 95 %.  Vector work of both products after both, in place of half after each,
// costs 3 %.  S_head 64, G = 1 (two workgroups per compute unit, 1 KB per product as before, but no hand-over): 4 x 1024 tokens, 16
// heads, bidirectional 89 -> 84; three to a unit want 168 registers and were slower.
template <int D, int G>
__global__ __launch_bounds__(256, G == 1 ? 2 : 1) void attn_bwd_dkv_wide_kernel(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ dctx,
                                                                   const float* __restrict__ lse, const float* __restrict__ delta,
                                                                   bf16_t* __restrict__ dqkv, int S_seq, int N_heads, int S_mb, int causal,
                                                                   float scale, float* __restrict__ colpart) {
  constexpr bool ASM = G == 2;
  constexpr int ROWS = 128 * G, NK = D / 16, NC = D / 16, PER = 2 * NK + 2 * NC, AHEAD = 3;  // steps of a score-sized product, of a gradient product, of a sub-tile
  __shared__ __attribute__((aligned(16))) bf16_t QOs[2][2][BLK * D];  // Q and dO tiles, double-buffered
  __shared__ __attribute__((aligned(16))) float stat_s[2][2][BLK];    // -lse log2(e) and -delta of the tile's queries
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);  // (uniform, and with it the loop over tiles)
  const int nhb = N_heads * S_mb;
  const int kblk = blockIdx.x / nhb;  // earliest keys see the most queries: those blocks of every head go first
  const int head = (blockIdx.x % nhb) % N_heads, b = (blockIdx.x % nhb) / N_heads;
  const int h = N_heads * D;
  const size_t ld = 3 * (size_t)h;
  const bf16_t* base = qkv + (size_t)b * S_seq * ld + head * D;
  const bf16_t* dob = dctx + (size_t)b * S_seq * h + head * D;
  const float* lrow = lse + ((size_t)b * N_heads + head) * S_seq;
  const float* drow = delta + ((size_t)b * N_heads + head) * S_seq;
  const int k0 = kblk * ROWS, kw = k0 + 32 * G * w;

  FragAddrX<D> fa;
  fa.init(lane);
  bf16x8 kf[G][D / 16], vf[G][D / 16];
  f32x16 dk[G][D / 32], dv[G][D / 32];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const bf16_t* row = base + (size_t)(kw + 32 * g + (lane & 31)) * ld;
    load_rowfrags<D>(row + h, lane, kf[g]);
    load_rowfrags<D>(row + 2 * h, lane, vf[g]);
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) { zero_acc<ASM>(dk[g][dt]); zero_acc<ASM>(dv[g][dt]); }
  }
  const float c2 = scale * LOG2E;
  const int jbeg = causal ? k0 / BLK : 0, nblk = S_seq / BLK;
  TileMover<D, D == 128 && G == 2 ? 2 : BLK * D / 8 / 256> mv;
  mv.init(base, 3 * h, dob, h, tid);
  const bool has_stat = tid < BLK;
  float lnext = 0.f, dnext = 0.f;
  auto next_stats = [&](int j) {
    if (has_stat) { lnext = -(lrow[j * BLK + tid] * LOG2E); dnext = -drow[j * BLK + tid]; }
  };
  auto store_stats = [&](int stage) {
    if (has_stat) { stat_s[stage][0][tid] = lnext; stat_s[stage][1][tid] = dnext; }
  };
  int cur = 0;  // LDS stage of the tile that is worked on
  next_stats(jbeg);
  mv.whole(jbeg, QOs[0][0]);
  store_stats(0);
  __syncthreads();

  // One query tile (whether it touches the diagonal is a compile-time constant); jn: the tile to be moved meanwhile
  auto body = [&](int j, int jn, auto diagc) {
    constexpr bool DIAG = decltype(diagc)::value;
    const bf16_t* Qs = QOs[0][0];  // the fragment offsets hold the stage
    const bf16_t* dOs = QOs[0][1];
    const float* st0 = stat_s[0][0] + cur * 2 * BLK + 4 * (lane >> 5);
    bf16_t* next = QOs[0][0] + (cur ^ 1) * 2 * BLK * D;
    const int qb = j * BLK;
    // fragment of step i (over both sub-tiles): S, dP, dV and dK of the first 32 queries, then of the others
    auto frag = [&](auto ic) {
      constexpr int i = decltype(ic)::value, t = i / PER, p = i % PER;
      if constexpr (p < NK) return fa.frag_k(Qs, 32 * t, p);
      else if constexpr (p < 2 * NK) return fa.frag_k(dOs, 32 * t, p - NK);
      else if constexpr (p < 2 * NK + NC) return fa.frag_t(dOs, 32 * t + 16 * ((p - 2 * NK) / (D / 32)), (p - 2 * NK) % (D / 32));
      else return fa.frag_t(Qs, 32 * t + 16 * ((p - 2 * NK - NC) / (D / 32)), (p - 2 * NK - NC) % (D / 32));
    };
    bf16x8 ring[AHEAD + 1];
    static_for<AHEAD>([&](auto ic) { ring[decltype(ic)::value] = frag(ic); });
    static_for<2>([&](auto tc) {
      constexpr int t = decltype(tc)::value;
      f32x16 s[G], dp[G];
      f32x4 nl[4], nd[4];        // -lse log2(e) and -delta of rows 4 q .. 4 q + 3, read two steps before their first use
      u32x4 pb[G][2], db[G][2];  // P and dS in bf16, rows 8 k .. 8 k + 7: the B operands of dV and dK
      // P = exp(S / sqrt(d) - lse) of row r
      auto exp_row = [&](int g, auto rc) {
        constexpr int r = decltype(rc)::value;
        float v = __builtin_amdgcn_exp2f(fmaf(s[g][r], c2, nl[r / 4][r % 4]));
        if (DIAG && kw + 32 * g + (lane & 31) > qb + 32 * t + acc_row(r, lane)) v = 0.f;
        s[g][r] = v;
        if constexpr (r % 2 == 1) pb[g][r / 8][r % 8 / 2] = pack2(s[g][r - 1], v);
      };
      // dS = P (dP - delta) (the factor 1/sqrt(d) is applied once, to dK; masked entries of P are zero)
      auto ds_row = [&](int g, auto rc) {
        constexpr int r = decltype(rc)::value;
        const uint32_t two = pb[g][r / 8][r % 8 / 2];
        dp[g][r] = __builtin_bit_cast(float, r % 2 ? two & 0xffff0000u : two << 16) * (dp[g][r] + nd[r / 4][r % 4]);
        if constexpr (r % 2 == 1) db[g][r / 8][r % 8 / 2] = pack2(dp[g][r - 1], dp[g][r]);
      };
      constexpr int RB = 10, H = NC / 2;  // dV and dK need rows 0-7 first
      // the step that takes row r first
      constexpr auto exp_step = [](int r) { return r < RB ? NK + ((r + 1) * NK - 1) / RB : 2 * NK + ((r + 1 - RB) * H - 1) / (16 - RB); };
      constexpr auto ds_step = [](int r) { return (r < 8 ? 2 * NK + H : 2 * NK + NC) + ((r % 8 + 1) * H - 1) / 8; };
      static_for<PER>([&](auto pc) {
        constexpr int p = decltype(pc)::value, i = t * PER + p;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (i + AHEAD < 2 * PER) ring[(i + AHEAD) % (AHEAD + 1)] = frag(std::integral_constant<int, i + AHEAD>{});
        const bf16x8 f = ring[i % (AHEAD + 1)];
        static_for<G>([&](auto gc) {  // a product, then vector work in its shadow
          constexpr int g = decltype(gc)::value;
          if constexpr (p < NK) {
            mfma_v<ASM>(s[g], f, kf[g][p], p == 0, DIAG);
          } else if constexpr (p < 2 * NK) {
            constexpr int k = p - NK;
            mfma_v<ASM>(dp[g], f, vf[g][k], k == 0, DIAG);
            __builtin_amdgcn_sched_barrier(0);
            share<0, RB, k, NK>([&](auto rc) { exp_row(g, rc); });
          } else if constexpr (p < 2 * NK + NC) {
            constexpr int c = p - 2 * NK;
            mfma_a<ASM>(dv[g][c % (D / 32)], f, __builtin_bit_cast(bf16x8, pb[g][c / (D / 32)]), DIAG || c % (D / 32) == 0);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (c < H) share<RB, 16, c, H>([&](auto rc) { exp_row(g, rc); });
            else share<0, 8, c - H, H>([&](auto rc) { ds_row(g, rc); });
          } else {
            constexpr int c = p - 2 * NK - NC;
            mfma_a<ASM>(dk[g][c % (D / 32)], f, __builtin_bit_cast(bf16x8, db[g][c / (D / 32)]), DIAG || c % (D / 32) == 0);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (c < H) share<8, 16, c, H>([&](auto rc) { ds_row(g, rc); });
          }
          __builtin_amdgcn_sched_barrier(0);
        });
        static_for<4>([&](auto qc) {
          constexpr int q = decltype(qc)::value;
          if constexpr (p == exp_step(4 * q) - 2) nl[q] = *reinterpret_cast<const f32x4*>(st0 + 32 * t + 8 * q);
          if constexpr (p == ds_step(4 * q) - 2) nd[q] = *reinterpret_cast<const f32x4*>(st0 + BLK + 32 * t + 8 * q);
        });
        mv.template step<i, 2 * PER>(jn, next);
      });
    });
    __builtin_amdgcn_sched_barrier(0);
  };
  auto end_tile = [&]() {
    store_stats(cur ^ 1);
    cur ^= 1;
    fa.flip(4 * BLK * D);
    __syncthreads();
  };
  // past the end the last tile is moved once more, which nobody reads
  int j = jbeg;
  if (causal) {
    // tiles whose queries are all before this wave's keys: it only moves its share of the next one
#pragma unroll 1
    for (; j * BLK + BLK - 1 < kw; ++j) {
      const int jn = min(j + 1, nblk - 1);
      next_stats(jn);
      mv.whole(jn, QOs[0][0] + (cur ^ 1) * 2 * BLK * D);
      end_tile();
    }
    const int jn = min(j + 1, nblk - 1);
    next_stats(jn);
    body(j, jn, std::true_type{});
    end_tile();
    ++j;
  }
#pragma unroll 1
  for (; j < nblk; ++j) {
    const int jn = min(j + 1, nblk - 1);
    next_stats(jn);
    body(j, jn, std::false_type{});
    end_tile();
  }
  if constexpr (ASM) drain();
  const int ln = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));  // (the lane again: no register holds it over the loop)
  // (the loop ended on a barrier; a sum is read out for the store and for its column sums at once)
  float* red = reinterpret_cast<float*>(&QOs[0][0][0]);
  float colscale = scale;
  asm("" : "+v"(colscale));  // (not the products that were stored: multiplied and added in one operation, as in the 128-key form)
#pragma unroll
  for (int g = 0; g < G; ++g) {
    bf16_t* out = dqkv + ((size_t)b * S_seq + kw + 32 * g + (ln & 31)) * ld + head * D;
    store_rows<D>(dk[g], out + h, ln, scale);
    if (colpart) wave_colsum<D>(dk[g], colscale, red + (size_t)(4 * G + w * G + g) * 4 * (D / 2), ln);
    store_rows<D>(dv[g], out + 2 * h, ln, 1.0f);
    if (colpart) wave_colsum<D>(dv[g], 1.0f, red + (size_t)(w * G + g) * 4 * (D / 2), ln);
  }
  if (colpart) {
    // rows (b, 128 keys) of the partial column sums of [dK | dV], [S_mb * S_seq / 128][2 N_heads * D], 32 keys at a time in order
    __syncthreads();
    for (int c = 64 * w + ln; c < 2 * D * G; c += 256) {
      const int blk = c / (2 * D), dvs = c / D % 2, d = c % D;
      colpart[((size_t)b * (S_seq / WG_ROWS) + kblk * G + blk) * 2 * h + dvs * h + head * D + d] = colsum_of<D>(red, (dvs ? 0 : 4 * G) + blk * 4, 4, d);
    }
  }
}

}  // namespace

// Which launches of S_head 128 go to 256-key workgroups.  A tile of those takes about 1.5 times as long as one of the 128-key
// form and covers twice the keys; a launch lasts as long as its longest block or its share per compute unit, whichever is more
// (rounds of equal blocks where nothing is masked), and the 128-key form's causal share comes out 1.12 times its tiles.
// Backward, 128- / 256-key form, us: causal, S_seq 2048, 32 heads 174 / 198, 40 210 / 207, 48 236 / 217, 64 302 / 266; 1024, 64
// heads 110 / 120, 80 132 / 128, 96 151 / 150; shorter rows never: 512, 160 heads 103 / 106, 256, 400 heads 111 / 114; 4096, 16
// heads 307 / 358, 24 415 / 393; bidirectional, 2048, 16 heads 160 / 200, 24 239 / 199, 64 521 / 441; 1024, 96 heads 243 / 248;
// 512, 300 heads 256 / 246; 256, 256 heads 71 / 64, 300 heads 108 / 110.  S_head 64, eight waves in pairs / here: 4 x 1024 tokens, 16 heads,
// bidirectional 89 / 84; 2048, 8 heads, causal 84 / 73; from S_seq 640 on 2 to 10 % less in launches of 32 to 1536 blocks of 128 keys, 512 1 to 5 %
// less, 384 level to 4 % less (causal, 768 blocks 2 % more).  Rows of two and four query tiles, most of whose time are the loads and stores at
// either end, better hidden by 16 waves to a unit than by 8: 128 3 to 4 % more up to 256 blocks, level above, 256 level up to 256, 1 to 4 % more above.
bool attention_bwd_dkv_wide_better(int S_mb, int S_seq, int N_heads, int S_head, int causal) {
  if (S_head == 64) return S_seq > 256;
  if (S_seq % 256 || (causal && S_seq < 1024)) return false;
  const double n = S_seq / 128, hb = (double)N_heads * S_mb;  // tiles of a whole block: 2 n
  double narrow, wide;
  if (causal) {
    narrow = 1.12 * std::max(2 * n, hb * n * (n + 1) / 256);
    wide = 1.55 * std::max(2 * n, hb * n * (n + 2) / 2 / 256);
  } else {
    narrow = 2 * n * std::ceil(hb * n / 256);
    wide = 1.55 * 2 * n * std::ceil(hb * n / 2 / 256);
  }
  return wide <= narrow;
}

bool attention_bwd_dkv_wide_supported(int S_mb, int S_seq, int N_heads, int S_head) {
  // 32-bit offsets inside a tile of 64 rows of 3 S_hidden
  return (S_head == 64 || (S_head == 128 && S_seq % 256 == 0)) && S_seq % 128 == 0 && (long)N_heads * S_head <= (1l << 22) && S_mb >= 1;
}

bf_status attention_bwd_dkv_wide(int S_mb, int S_seq, int N_heads, int S_head, int causal, const void* qkv, const float* lse, const void* dctx,
                                 void* dqkv, const float* delta, float* part_kv, hipStream_t st) {
  if (!attention_bwd_dkv_wide_supported(S_mb, S_seq, N_heads, S_head)) { set_error("attention_bwd_dkv_wide: shape not supported"); return BF_EINVAL; }
  const float scale = 1.0f / sqrtf((float)S_head);
  const unsigned grid = (unsigned)(S_seq / (S_head == 128 ? 256 : 128)) * N_heads * S_mb;
  if (S_head == 128)
    attn_bwd_dkv_wide_kernel<128, 2><<<grid, 256, 0, st>>>((const bf16_t*)qkv, (const bf16_t*)dctx, lse, delta, (bf16_t*)dqkv, S_seq, N_heads, S_mb, causal, scale, part_kv);
  else
    attn_bwd_dkv_wide_kernel<64, 1><<<grid, 256, 0, st>>>((const bf16_t*)qkv, (const bf16_t*)dctx, lse, delta, (bf16_t*)dqkv, S_seq, N_heads, S_mb, causal, scale, part_kv);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_error("attention_bwd_dkv_wide launch failed: %s", hipGetErrorString(e)); return BF_EDEVICE; }
  return BF_OK;
}


}  // namespace bf
