// float32 kernels on the bfloat16 matrix cores: every operand is split into
// three bfloat16 parts, x = hi + mid + lo (8 + 8 + 8 significand bits, each
// part rounded to nearest, so that nothing of an x of 2^-110 or more is lost;
// below, lo falls under the smallest bfloat16), and a product is the six
// part products down to 2^-16 of the largest (hi hi, hi mid, mid hi, mid mid,
// hi lo, lo hi), accumulated in float32, the small ones first. What is left
// out (mid lo, lo mid, lo lo) is below 2^-25 of a product, less than the
// rounding of one float32 addition. A float32 product on the matrix cores runs
// at 1/16 of the bfloat16 rate, so six cost 0.375 of one. Softmax, dS and all
// sums stay in float32.
//
// Infinities do not split, nor do values below 2^-110 other than 0, and part
// products of large values overflow on their own (Range). Every tile and a
// wave's own rows are tested for such values, and a workgroup that meets one goes
// on from that tile with float32 matrix instructions, on tiles stored as they are
// in the LDS of the parts. Accumulators that hold an infinity or NaN after the
// fast tiles, which P or dS beyond the range leave there (attn_bwd takes any L and
// O), are formed again that way. Results are those of float32 arithmetic then.
//
// (The decomposition into bfloat16 parts is the one of Henry, Tang and Heinecke,
// "Leveraging the bfloat16 Artificial Intelligence Datatype For Higher-Precision
// Computations", 2019: three parts, six products.)
//
// Measured (us, float32 matrix instructions / these; MI355X): 64 heads, n =
// 2048, d = 64: forward 557 / 399, dK/dV 1189 / 715, dQ 892 / 523; d = 32: 289 / 245,
// 558 / 421, 427 / 313; d = 128: 1349 / 789, 2613 / 1545, 1793 / 1189; 32 heads, n =
// 1024, d = 64: 86 / 61, 159 / 103, 120 / 77. The tests for values that do not split,
// the scaling of P and dS and the test of the accumulators are 2.5 % of that.
// Relative error against float64 over n = 128 to 8192 and sigma 1 and 2: 0.5 to 1.0
// of what it was (a product's 16 terms are added before they are rounded, where
// the float32 instruction rounds every 2).
// Bound by the matrix cores and the power they draw (1070 to 1200 TFLOP/s of
// bfloat16 products, what a large bfloat16 matrix product reaches), then by
// the VALU work of the splits. With keys masked by -inf or by large values (64
// heads, n = 2048, d = 64; a quarter of the keys, every eighth): forward 546 on the
// float32 instructions throughout, 417 and 541 here; d = 128, 32 heads, n = 1024:
// 175, 145 and 164; worst at d = 32 without a mask, every eighth key: 77 and 91.
//
// Tiles are read from memory as float32, a tile ahead, into registers, split
// once, and written to LDS as three bfloat16 tiles in the layouts of RowRead
// and TransRead. P and dS are split in registers.
#pragma once

#include "kernels.hpp"

namespace attn {

typedef float f32x8 __attribute__((ext_vector_type(8)));

struct Parts {
  bf16x8 hi, mid, lo;
};
__device__ __forceinline__ Parts split3(const f32x8& x) {
  Parts p;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    p.hi[i] = (bf16)x[i];
    const float r = x[i] - (float)p.hi[i];
    p.mid[i] = (bf16)r;
    p.lo[i] = (bf16)(r - (float)p.mid[i]);
  }
  return p;
}
__device__ __forceinline__ Parts split3(const f32x16& v, int t) {
  f32x8 x;
#pragma unroll
  for (int i = 0; i < 8; ++i) x[i] = v[8 * t + i];
  return split3(x);
}
// P and dS, whose small values are ordinary, are formed 2^24 times as large and
// the accumulators scaled back at the end: all of their normal values (2^-126 on)
// then split without loss, and dS's subnormal ones too. (The matrix cores take and
// give subnormals.)
constexpr float kUp = 0x1p24f, kDown = 0x1p-24f;
// Whether values split: 0, or kSplitMin <= |x| < kSplitMax. Under kSplitMax
// neither part products nor what the kernels form from them leave the float32
// range: scores and dP stay below 2^55, dS, with P <= 1, below 2^57, 2^24 dS
// below 2^81, and sums of it over 2^20 rows below 2^125. From there on a product
// can overflow while a part product of the other sign does too, to NaN where
// float32 arithmetic gives an infinity.
struct Range {
  static constexpr float kSplitMax = 0x1p24f;
  static constexpr uint32_t kSplitMin = 17u << 23;   // bits of 2^-110
  float mx = 0.f;
  uint32_t mn = ~0u;   // least 2 bits(|x|) - 1, of which 0 gives the largest
  __device__ __forceinline__ void add(const f32x8& x) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      mx = fmaxf(mx, fabsf(x[i]));
      mn = min(mn, (__float_as_uint(x[i]) << 1) - 1u);
    }
  }
  // whether a lane of the wave has met a value that does not split
  __device__ __forceinline__ bool left() const {
    return __builtin_amdgcn_ballot_w64(mx >= kSplitMax || mn < 2u * kSplitMin - 1u) != 0;
  }
};
__device__ __forceinline__ void mma6(f32x16& acc, const Parts& a, const Parts& b) {
  mma(acc, a.lo, b.hi);
  mma(acc, a.hi, b.lo);
  mma(acc, a.mid, b.mid);
  mma(acc, a.mid, b.hi);
  mma(acc, a.hi, b.mid);
  mma(acc, a.hi, b.hi);
}

__device__ __forceinline__ f32x8 as_f32x8(u32x4 a, u32x4 b) {
  f32x8 x;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    x[e] = __uint_as_float(a[e]);
    x[4 + e] = __uint_as_float(b[e]);
  }
  return x;
}

// Row operands of one row per lane: k-step t holds columns 16t + 8h + [0, 8).
// load() returns whether the wave's rows hold something that does not split,
// and takes a power of two to multiply the rows by.
template <int D> struct RowParts {
  Parts f[D / 16];
  __device__ __forceinline__ bool load(const float* g, int row, int n, int h, uint32_t flip, float up = 1.f) {
    f32x8 x[D / 16];
    Range m;
#pragma unroll
    for (int t = 0; t < D / 16; ++t) {
      u32x4 a = {0u, 0u, 0u, 0u}, b = a;
      if (row < n) {
        const u32x4* p = (const u32x4*)(g + (size_t)row * D + 16 * t + 8 * h);
        a = p[0] ^ (u32x4){flip, flip, flip, flip};
        b = p[1] ^ (u32x4){flip, flip, flip, flip};
      }
      x[t] = as_f32x8(a, b);
      m.add(x[t]);
    }
#pragma unroll
    for (int t = 0; t < D / 16; ++t) f[t] = split3(x[t] * up);
    return m.left();
  }
};

// A ROWS x D tile on its way from memory to three LDS tiles, by NT threads.
// Rows >= n are zeros.
template <int ROWS, int D, int NT> struct Stage3 {
  static constexpr int C = D / 8, NCH = ROWS * C, NPT = NCH / NT, ELEMS = ROWS * D;
  static_assert(NCH % NT == 0, "whole 8-element chunks per thread");
  u32x4 r[NPT][2];
  __device__ __forceinline__ void load(const float* g, int row0, int n, int tid) {
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
      const int ci = tid + NT * i, row = row0 + ci / C;
      r[i][0] = r[i][1] = (u32x4){0u, 0u, 0u, 0u};
      if (row < n) {
        const u32x4* p = (const u32x4*)(g + (size_t)row * D + 8 * (ci % C));
        r[i][0] = p[0];
        r[i][1] = p[1];
      }
    }
  }
  __device__ __forceinline__ static void put(bf16* lds, int ci, const Parts& p) {
    const int s = srow(ci / C);
    bf16* o = lds + s * D + 8 * ((ci % C) ^ swz<D>(s));
    *(bf16x8*)o = p.hi;
    *(bf16x8*)(o + ELEMS) = p.mid;
    *(bf16x8*)(o + 2 * ELEMS) = p.lo;
  }
  // returns whether the wave's part holds something that does not split
  __device__ __forceinline__ bool store(bf16* lds, int tid) const {
    Range m;
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
      const f32x8 x = as_f32x8(r[i][0], r[i][1]);
      m.add(x);
      put(lds, tid + NT * i, split3(x));
    }
    return m.left();
  }
  // the tile as it is, in the layout of RowRead<float> and TransRead<float>
  __device__ __forceinline__ void store_f32(float* lds, int tid) const {
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
      const int ci = tid + NT * i;
      float* o = lds + srow(ci / C) * Tile<float, ROWS, D>::LD + 8 * (ci % C);
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = __uint_as_float(r[i][e / 4][e % 4]);
    }
  }
};
// The float32 products, on tiles stored as they are (Stage3::store_f32).
template <int D>
__device__ __forceinline__ void rows_f32(f32x16& acc, const float* tile, int rb, const RowFrags<float, D>& b, int h, int c) {
#pragma unroll
  for (int t = 0; t < D / 2; ++t) mma(acc, RowRead<float, D>::get(tile, rb, t, h, c), b.f[t]);
}
template <int D, int ROWS>
__device__ __forceinline__ void cols_f32(f32x16 (&acc)[D / 32], const float* tile, int rb, const f32x16& b, int h, int c) {
#pragma unroll
  for (int t = 0; t < 16; ++t)
#pragma unroll
    for (int db = 0; db < D / 32; ++db) mma(acc[db], TransRead<float, D, ROWS>::get(tile, rb, db, t, h, c), b[t]);
}
// whether any of the NW waves set its flag
template <int NW> __device__ __forceinline__ bool any_flag(const int (&f)[NW]) {
  int r = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) r |= f[i];
  return __builtin_amdgcn_readfirstlane(r) != 0;
}
// whether an accumulator of this wave holds an infinity or NaN
template <int N> __device__ __forceinline__ bool any_nonfinite(const f32x16 (&a)[N]) {
  float x = 0.f;
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < 16; ++j) x = fmaf(a[i][j], 0.f, x);
  return __builtin_amdgcn_ballot_w64(x != 0.f) != 0;   // NaN from either
}
// whether any wave of the workgroup has `f`
template <int NW> __device__ __forceinline__ bool any_wave(int (&flag)[NW], int wv, int lane, bool f) {
  if (lane == 0) flag[wv] = f;
  __syncthreads();
  return any_flag(flag);
}
template <int D, int ROWS> __device__ __forceinline__ Parts row_parts(const bf16* s, int rb, int t, int h, int c) {
  return {RowRead<bf16, D>::get(s, rb, t, h, c), RowRead<bf16, D>::get(s + ROWS * D, rb, t, h, c),
          RowRead<bf16, D>::get(s + 2 * ROWS * D, rb, t, h, c)};
}
template <int D, int ROWS> __device__ __forceinline__ Parts col_parts(const bf16* s, int rb, int db, int t, int h, int c) {
  return {TransRead<bf16, D, ROWS>::get(s, rb, db, t, h, c), TransRead<bf16, D, ROWS>::get(s + ROWS * D, rb, db, t, h, c),
          TransRead<bf16, D, ROWS>::get(s + 2 * ROWS * D, rb, db, t, h, c)};
}

// ======================================================================
// Forward: 128 queries, 32 per wave, key tiles of BT rows. KS = 2: two groups
// of four waves own the same queries and take the two halves of every tile,
// merged by log-sum-exp at the end.
// ======================================================================
template <int D, bool CAUSAL, int KS, int BT>
__global__ void __launch_bounds__(256 * KS, 2) fwd_x3_kernel(const FwdArgs a) {
  constexpr int NT = 256 * KS, NB = BT / 32 / KS, NDB = D / 32;
  using ST = Stage3<BT, D, NT>;
  constexpr int MERGE = KS == 2 ? 4 * 64 * (16 * NDB + 2) * 4 : 0;   // bytes
  constexpr int TILES = 2 * 3 * ST::ELEMS * 2;
  using TF = Tile<float, BT, D>;
  static_assert(2 * TF::ELEMS * 4 <= TILES, "the float32 tiles go where the parts went");
  __shared__ __attribute__((aligned(16))) bf16 st[(TILES > MERGE ? TILES : MERGE) / 2];
  __shared__ int flag[4 * KS];   // per wave: its part of the tile does not split
  __shared__ int bad[4 * KS];    // per wave: its accumulators are not finite
  bf16* const kl = st;
  bf16* const vl = st + 3 * ST::ELEMS;

  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, c = lane & 31;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), w = wv & 3, ks = wv >> 2;
  int head, qt;
  block_map(blockIdx.x, a.nblocks, a.ntiles, CAUSAL ? a.hgroup : 0, CAUSAL, head, qt);
  const int n = a.n;
  const size_t hoff = (size_t)head * (size_t)a.head_stride;
  const float* Kg = (const float*)a.k + hoff;
  const float* Vg = (const float*)a.v + hoff;
  const int q0 = 128 * qt, qw0 = q0 + 32 * w, qi = qw0 + c;
  const int nt = ((CAUSAL ? min(n, q0 + 128) : n) + BT - 1) / BT;

  ST ksg, vsg;
  ksg.load(Kg, 0, n, tid);
  vsg.load(Vg, 0, n, tid);
  const float* Qg = (const float*)a.q + hoff;
  RowParts<D> q;
  const bool own = q.load(Qg, qi, n, h, a.qflip);

  f32x16 oacc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) oacc[db] = zero16();
  float m_use = -INFINITY, lsum = 0.f;
  const float sl2 = a.sl2;
  // scores of the keys from kv0 on -> up P, moving the running maximum and sum
  auto softmax = [&](int kv0, auto& s, float up) __attribute__((always_inline)) {
    constexpr int B = sizeof(s) / sizeof(f32x16);
    if (kv0 + 32 * B > n || (CAUSAL && kv0 + 32 * B - 1 > qw0)) {
      const int last = CAUSAL ? min(qi, n - 1) : n - 1;
#pragma unroll
      for (int b = 0; b < B; ++b) {
        const int lim = last - (kv0 + 32 * b + 16 * h);
#pragma unroll
        for (int j = 0; j < 16; ++j) s[b][j] = (j > lim) ? -INFINITY : s[b][j];
      }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int b = 0; b < B; ++b)
#pragma unroll
      for (int j = 0; j < 16; ++j) mx = fmaxf(mx, s[b][j]);
    const float mt = halves_max(mx) * sl2;
    const bool resc = mt > m_use + kRescaleThresh;
    if (__builtin_amdgcn_ballot_w64(resc)) {
      const float alpha = resc ? exp2_fast(m_use - mt) : 1.f;
      if (resc) m_use = mt;
      lsum *= alpha;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int j = 0; j < 16; ++j) oacc[db][j] *= alpha;
    }
    const float mb = (m_use == -INFINITY) ? 0.f : -m_use;
    float rs = 0.f;   // a tile's sum first: thousands of single terms would lose bits in lsum
#pragma unroll
    for (int b = 0; b < B; ++b)
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        s[b][j] = exp2_fast(fmaf(s[b][j], sl2, mb)) * up;
        rs += s[b][j];
      }
    lsum += rs;
  };

  bool slow = false;   // from tile `it` on
  int it = 0;
  for (; it < nt; ++it) {
    const int t0 = it * BT, kv0 = t0 + 32 * NB * ks;   // this group's first key
    __syncthreads();
    const bool huge_k = ksg.store(kl, tid), huge_v = vsg.store(vl, tid);
    if (lane == 0) flag[wv] = own || huge_k || huge_v;
    __syncthreads();
    if ((slow = any_flag(flag))) break;
    if (it + 1 < nt) {
      ksg.load(Kg, t0 + BT, n, tid);
      vsg.load(Vg, t0 + BT, n, tid);
    }
    if (kv0 >= n || (CAUSAL && kv0 > qw0 + 31)) continue;
    f32x16 s[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) s[b] = zero16();
#pragma unroll
    for (int t = 0; t < D / 16; ++t)
#pragma unroll
      for (int b = 0; b < NB; ++b) mma6(s[b], row_parts<D, BT>(kl, NB * ks + b, t, h, c), q.f[t]);
    softmax(kv0, s, kUp);
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const Parts p = split3(s[b], t);
#pragma unroll
        for (int db = 0; db < NDB; ++db) mma6(oacc[db], col_parts<D, BT>(vl, NB * ks + b, db, t, h, c), p);
      }
  }

  __builtin_amdgcn_sched_barrier(0);   // keeps the test out of the loop's schedule (35 more spills without)
  float down = kDown;
  if (any_wave(bad, wv, lane, any_nonfinite(oacc))) {   // all over again
    slow = true, it = 0, down = 0.f;
    m_use = -INFINITY;
    ksg.load(Kg, 0, n, tid);
    vsg.load(Vg, 0, n, tid);
  }
  lsum = down == 0.f ? 0.f : lsum * down;
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int j = 0; j < 16; ++j) oacc[db][j] = down == 0.f ? 0.f : oacc[db][j] * down;
  if (slow) {
    RowFrags<float, D> qf;
    qf.load(Qg, qi, n, h, a.qflip);
    float* const kf = (float*)st;
    float* const vf = kf + TF::ELEMS;
#pragma unroll 1
    for (; it < nt; ++it) {
      const int t0 = it * BT;
      __syncthreads();
      ksg.store_f32(kf, tid);
      vsg.store_f32(vf, tid);
      __syncthreads();
      if (it + 1 < nt) {
        ksg.load(Kg, t0 + BT, n, tid);
        vsg.load(Vg, t0 + BT, n, tid);
      }
      const int kv0 = t0 + 32 * NB * ks;
      if (kv0 >= n || (CAUSAL && kv0 > qw0 + 31)) continue;
      f32x16 s[NB];
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        s[b] = zero16();
        rows_f32<D>(s[b], kf, NB * ks + b, qf, h, c);
      }
      softmax(kv0, s, 1.f);
#pragma unroll
      for (int b = 0; b < NB; ++b) cols_f32<D, BT>(oacc, vf, NB * ks + b, s[b], h, c);
    }
  }

  float ltot = halves_sum(lsum);
  if constexpr (KS == 2) {
    // the second group's (max, sum, O) into the first's
    float* mg = (float*)st + w * 64 * (16 * NDB + 2) + lane;
    __syncthreads();
    if (ks == 1) {
      mg[0] = m_use;
      mg[64] = ltot;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int j = 0; j < 16; ++j) mg[64 * (2 + 16 * db + j)] = oacc[db][j];
    }
    __syncthreads();
    if (ks == 1) return;
    const float m1 = mg[0], M = fmaxf(m_use, m1);
    const float f0 = (M == -INFINITY) ? 0.f : exp2_fast(m_use - M), f1 = (M == -INFINITY) ? 0.f : exp2_fast(m1 - M);
    ltot = f0 * ltot + f1 * mg[64];
    m_use = M;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int j = 0; j < 16; ++j) oacc[db][j] = f0 * oacc[db][j] + f1 * mg[64 * (2 + 16 * db + j)];
  }

  // ---- epilogue: lane (h, c) holds O^T columns of query qi
  const float inv = 1.f / ltot;
  float* Og = (float*)a.o + hoff;
  const float* dOg = a.dout ? (const float*)a.dout + hoff : nullptr;
  float dpart = 0.f;
  if (qi < n) {
#pragma unroll
    for (int db = 0; db < NDB; ++db) {
      f32x4 g[4];
      if (dOg) {
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) g[q4] = *(const f32x4*)(dOg + (size_t)qi * D + 32 * db + 8 * q4 + 4 * h);
      }
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        f32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          o[e] = oacc[db][4 * q4 + e] * inv;
          if (dOg) dpart += o[e] * g[q4][e];
        }
        *(f32x4*)(Og + (size_t)qi * D + 32 * db + 8 * q4 + 4 * h) = o;
      }
    }
  }
  const float dsum = halves_sum(dpart);
  if (qi < n && h == 0) {
    const size_t row = (size_t)head * n + qi;
    const float l2 = m_use + log2f(ltot);
    a.lse[row] = l2 * kLn2;
    if (dOg) {
      a.dvec[row] = -dsum;   // stored negated (the backward starts dP - D from it)
      a.lse2[row] = l2;
    }
  }
}

// ======================================================================
// dQ: 128 queries, 32 per wave (Q and dO parts in registers), key tiles of BT
// rows; KS as in the forward, the two groups' dQ added.
// ======================================================================
template <int D, bool CAUSAL, int KS, int BT>
__global__ void __launch_bounds__(256 * KS, D == 128 ? 1 : 2) dq_x3_kernel(const BwdArgs a) {
  constexpr int NT = 256 * KS, NB = BT / 32 / KS, NDB = D / 32;
  using ST = Stage3<BT, D, NT>;
  constexpr int MERGE = KS == 2 ? 4 * 64 * 16 * NDB * 4 : 0;   // bytes
  constexpr int TILES = 2 * 3 * ST::ELEMS * 2;
  using TF = Tile<float, BT, D>;
  static_assert(2 * TF::ELEMS * 4 <= TILES, "the float32 tiles go where the parts went");
  __shared__ __attribute__((aligned(16))) bf16 st[(TILES > MERGE ? TILES : MERGE) / 2];
  __shared__ int flag[4 * KS];   // per wave: its part of the tile does not split
  __shared__ int bad[4 * KS];    // per wave: its accumulators are not finite
  bf16* const kl = st;
  bf16* const vl = st + 3 * ST::ELEMS;

  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, c = lane & 31;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), w = wv & 3, ks = wv >> 2;
  int head, qt;
  block_map(blockIdx.x, a.nblocks, a.ntiles, CAUSAL ? a.hgroup : 0, CAUSAL, head, qt);
  const int n = a.n;
  const size_t hoff = (size_t)head * (size_t)a.head_stride;
  const float* Kg = (const float*)a.k + hoff;
  const float* Vg = (const float*)a.v + hoff;
  const int q0 = 128 * qt, qw0 = q0 + 32 * w, qi = qw0 + c;
  const int nt = ((CAUSAL ? min(n, q0 + 128) : n) + BT - 1) / BT;

  ST ksg, vsg;
  ksg.load(Kg, 0, n, tid);
  vsg.load(Vg, 0, n, tid);
  const float* Qg = (const float*)a.q + hoff;
  const float* dOg = (const float*)a.dout + hoff;
  RowParts<D> q, g;
  // dO and D 2^24 times as large, so that dS is
  const bool own_q = q.load(Qg, qi, n, h, a.qflip), own_g = g.load(dOg, qi, n, h, 0u, kUp), own = own_q || own_g;
  const float lq = qi < n ? a.lse2[(size_t)head * n + qi] : 0.f;
  const float nd = qi < n ? a.dvec[(size_t)head * n + qi] : 0.f;   // -D

  f32x16 dqa[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) dqa[db] = zero16();
  const float sl2 = a.sl2;
  // dS of the 32 keys from kv0 on, from S and dP (which becomes dS)
  auto grad = [&](int kv0, const f32x16& s, f32x16& dp, float nd) __attribute__((always_inline)) {
    const bool edge = kv0 + 32 > n || (CAUSAL && kv0 + 31 > qw0);
    const int lim = (CAUSAL ? min(qi, n - 1) : n - 1) - (kv0 + 16 * h);
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      float p = exp2_fast(fmaf(s[j], sl2, -lq));
      if (edge) p = (j > lim) ? 0.f : p;
      dp[j] = p * (dp[j] + nd);
    }
  };

  bool slow = false;   // from tile `it` on
  int it = 0;
  for (; it < nt; ++it) {
    const int t0 = it * BT;
    __syncthreads();
    const bool huge_k = ksg.store(kl, tid), huge_v = vsg.store(vl, tid);
    if (lane == 0) flag[wv] = own || huge_k || huge_v;
    __syncthreads();
    if ((slow = any_flag(flag))) break;
    if (it + 1 < nt) {
      ksg.load(Kg, t0 + BT, n, tid);
      vsg.load(Vg, t0 + BT, n, tid);
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int rb = NB * ks + b, kv0 = t0 + 32 * rb;
      if (kv0 >= n || (CAUSAL && kv0 > qw0 + 31)) continue;
      f32x16 s = zero16(), dp = zero16();
#pragma unroll
      for (int t = 0; t < D / 16; ++t) {
        mma6(s, row_parts<D, BT>(kl, rb, t, h, c), q.f[t]);
        mma6(dp, row_parts<D, BT>(vl, rb, t, h, c), g.f[t]);
      }
      grad(kv0, s, dp, nd * kUp);
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const Parts f = split3(dp, t);
#pragma unroll
        for (int db = 0; db < NDB; ++db) mma6(dqa[db], col_parts<D, BT>(kl, rb, db, t, h, c), f);
      }
    }
  }

  __builtin_amdgcn_sched_barrier(0);   // keeps the test out of the loop's schedule (35 more spills without)
  float down = kDown;
  if (any_wave(bad, wv, lane, any_nonfinite(dqa))) {   // all over again
    slow = true, it = 0, down = 0.f;
    ksg.load(Kg, 0, n, tid);
    vsg.load(Vg, 0, n, tid);
  }
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int j = 0; j < 16; ++j) dqa[db][j] = down == 0.f ? 0.f : dqa[db][j] * down;
  if (slow) {
    RowFrags<float, D> qf, gf;
    qf.load(Qg, qi, n, h, a.qflip);
    gf.load(dOg, qi, n, h, 0u);
    float* const kf = (float*)st;
    float* const vf = kf + TF::ELEMS;
#pragma unroll 1
    for (; it < nt; ++it) {
      const int t0 = it * BT;
      __syncthreads();
      ksg.store_f32(kf, tid);
      vsg.store_f32(vf, tid);
      __syncthreads();
      if (it + 1 < nt) {
        ksg.load(Kg, t0 + BT, n, tid);
        vsg.load(Vg, t0 + BT, n, tid);
      }
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int rb = NB * ks + b, kv0 = t0 + 32 * rb;
        if (kv0 >= n || (CAUSAL && kv0 > qw0 + 31)) continue;
        f32x16 s = zero16(), dp = zero16();
        rows_f32<D>(s, kf, rb, qf, h, c);
        rows_f32<D>(dp, vf, rb, gf, h, c);
        grad(kv0, s, dp, nd);
        cols_f32<D, BT>(dqa, kf, rb, dp, h, c);
      }
    }
  }

  if constexpr (KS == 2) {
    float* mg = (float*)st + w * 64 * 16 * NDB + lane;
    __syncthreads();
    if (ks == 1) {
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int j = 0; j < 16; ++j) mg[64 * (16 * db + j)] = dqa[db][j];
    }
    __syncthreads();
    if (ks == 1) return;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int j = 0; j < 16; ++j) dqa[db][j] += mg[64 * (16 * db + j)];
  }
  if (qi < n) {
    float* out = (float*)a.dq + hoff + (size_t)qi * D;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        Quad<float>::store(out + 32 * db + 8 * q4 + 4 * h, dqa[db][4 * q4] * a.dq_scale, dqa[db][4 * q4 + 1] * a.dq_scale,
                           dqa[db][4 * q4 + 2] * a.dq_scale, dqa[db][4 * q4 + 3] * a.dq_scale);
  }
}

// ======================================================================
// dK, dV: 128 keys, 32 per wave (K and V parts in registers), query tiles of
// BT rows with their base-2 log-sum-exp and -D; KS as in the forward, the two
// groups' dK and dV added.
// ======================================================================
template <int D, bool CAUSAL, int KS, int BT>
__global__ void __launch_bounds__(256 * KS, D == 128 ? 1 : 2) dkdv_x3_kernel(const BwdArgs a) {
  constexpr int NT = 256 * KS, NB = BT / 32 / KS, NDB = D / 32;
  using ST = Stage3<BT, D, NT>;
  constexpr int MERGE = KS == 2 ? 4 * 64 * 16 * NDB * 4 : 0;   // bytes
  constexpr int TILES = 2 * 3 * ST::ELEMS * 2;
  using TF = Tile<float, BT, D>;
  static_assert(2 * TF::ELEMS * 4 <= TILES, "the float32 tiles go where the parts went");
  __shared__ __attribute__((aligned(16))) bf16 st[(TILES > MERGE ? TILES : MERGE) / 2];
  __shared__ int flag[4 * KS];   // per wave: its part of the tile does not split
  __shared__ int bad[4 * KS];    // per wave: its accumulators are not finite
  __shared__ __attribute__((aligned(16))) float ld[2][BT];   // the tile's L and -D rows
  bf16* const ql = st;
  bf16* const ol = st + 3 * ST::ELEMS;

  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, c = lane & 31;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), w = wv & 3, ks = wv >> 2;
  int head, kt;
  block_map(blockIdx.x, a.nblocks, a.ntiles, CAUSAL ? a.hgroup : 0, false, head, kt);
  const int n = a.n;
  const size_t hoff = (size_t)head * (size_t)a.head_stride;
  const float* Qg = (const float*)a.q + hoff;
  const float* dOg = (const float*)a.dout + hoff;
  const float* Lg = a.lse2 + (size_t)head * n;
  const float* Dg = a.dvec + (size_t)head * n;
  const int k0 = 128 * kt, kw0 = k0 + 32 * w, kj = kw0 + c;
  const int q_begin = CAUSAL ? k0 / BT * BT : 0;
  const int nt = (n - q_begin + BT - 1) / BT;

  ST qsg, osg;
  float lr = 0.f;   // thread t < 2 BT: one element of the L, then the -D rows
  auto load = [&](int r0) __attribute__((always_inline)) {
    qsg.load(Qg, r0, n, tid);
    osg.load(dOg, r0, n, tid);
    if (tid < 2 * BT) lr = (tid < BT ? Lg : Dg)[min(r0 + tid % BT, n - 1)];
  };
  load(q_begin);
  RowParts<D> k, v;   // K sign-flipped for a negative scale
  const float* Kg = (const float*)a.k + hoff;
  const float* Vg = (const float*)a.v + hoff;
  const bool own_k = k.load(Kg, kj, n, h, a.qflip), own_v = v.load(Vg, kj, n, h, 0u), own = own_k || own_v;

  f32x16 dk[NDB], dv[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) { dk[db] = zero16(); dv[db] = zero16(); }
  const float sl2 = a.sl2;
  // up P (in s) and up dS (in dp) of the tile's 32 queries from qb0 on, from S and
  // dP; lane (h, c): element j is query qb0 + 16h + j, key kj
  auto grad = [&](int rb, int qb0, f32x16& s, f32x16& dp, float up) __attribute__((always_inline)) {
    const bool edge = qb0 + 32 > n || (CAUSAL && qb0 < kw0 + 31);
    const int qbase = qb0 + 16 * h, lo = CAUSAL ? kj - qbase : -1, hi = n - 1 - qbase;
#pragma unroll
    for (int j4 = 0; j4 < 4; ++j4) {
      const f32x4 l4 = *(const f32x4*)&ld[0][32 * rb + 16 * h + 4 * j4];
      const f32x4 d4 = *(const f32x4*)&ld[1][32 * rb + 16 * h + 4 * j4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = 4 * j4 + e;
        float p = exp2_fast(fmaf(s[j], sl2, -l4[e])) * up;
        if (edge) p = (j < lo || j > hi) ? 0.f : p;
        s[j] = p;
        dp[j] = p * (dp[j] + d4[e]);   // d4 holds -D
      }
    }
  };

  bool slow = false;   // from tile `it` on
  int it = 0;
  for (; it < nt; ++it) {
    const int t0 = q_begin + it * BT;
    __syncthreads();
    const bool huge_q = qsg.store(ql, tid), huge_o = osg.store(ol, tid);
    if (lane == 0) flag[wv] = own || huge_q || huge_o;
    if (tid < 2 * BT) (&ld[0][0])[tid] = lr;
    __syncthreads();
    if ((slow = any_flag(flag))) break;
    if (it + 1 < nt) load(t0 + BT);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int rb = NB * ks + b, qb0 = t0 + 32 * rb;
      if (qb0 >= n || (CAUSAL && qb0 + 31 < kw0)) continue;
      f32x16 s = zero16(), dp = zero16();
#pragma unroll
      for (int t = 0; t < D / 16; ++t) {
        mma6(s, row_parts<D, BT>(ql, rb, t, h, c), k.f[t]);
        mma6(dp, row_parts<D, BT>(ol, rb, t, h, c), v.f[t]);
      }
      grad(rb, qb0, s, dp, kUp);
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const Parts pf = split3(s, t);
#pragma unroll
        for (int db = 0; db < NDB; ++db) mma6(dv[db], col_parts<D, BT>(ol, rb, db, t, h, c), pf);
        const Parts sf = split3(dp, t);
#pragma unroll
        for (int db = 0; db < NDB; ++db) mma6(dk[db], col_parts<D, BT>(ql, rb, db, t, h, c), sf);
      }
    }
  }

  __builtin_amdgcn_sched_barrier(0);   // keeps the test out of the loop's schedule (35 more spills without)
  float down = kDown;
  if (any_wave(bad, wv, lane, any_nonfinite(dk) || any_nonfinite(dv))) {   // all over again
    slow = true, it = 0, down = 0.f;
    load(q_begin);
  }
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      dk[db][j] = down == 0.f ? 0.f : dk[db][j] * down;
      dv[db][j] = down == 0.f ? 0.f : dv[db][j] * down;
    }
  if (slow) {
    RowFrags<float, D> kf, vf;
    kf.load(Kg, kj, n, h, a.qflip);
    vf.load(Vg, kj, n, h, 0u);
    float* const qt = (float*)st;
    float* const ot = qt + TF::ELEMS;
#pragma unroll 1
    for (; it < nt; ++it) {
      const int t0 = q_begin + it * BT;
      __syncthreads();
      qsg.store_f32(qt, tid);
      osg.store_f32(ot, tid);
      if (tid < 2 * BT) (&ld[0][0])[tid] = lr;
      __syncthreads();
      if (it + 1 < nt) load(t0 + BT);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int rb = NB * ks + b, qb0 = t0 + 32 * rb;
        if (qb0 >= n || (CAUSAL && qb0 + 31 < kw0)) continue;
        f32x16 s = zero16(), dp = zero16();
        rows_f32<D>(s, qt, rb, kf, h, c);
        rows_f32<D>(dp, ot, rb, vf, h, c);
        grad(rb, qb0, s, dp, 1.f);
        cols_f32<D, BT>(dv, ot, rb, s, h, c);
        cols_f32<D, BT>(dk, qt, rb, dp, h, c);
      }
    }
  }

  auto finish = [&](f32x16 (&acc)[NDB], void* outp, float sc) __attribute__((always_inline)) {
    if constexpr (KS == 2) {
      float* mg = (float*)st + w * 64 * 16 * NDB + lane;
      __syncthreads();
      if (ks == 1) {
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
          for (int j = 0; j < 16; ++j) mg[64 * (16 * db + j)] = acc[db][j];
      }
      __syncthreads();
      if (ks == 0) {
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
          for (int j = 0; j < 16; ++j) acc[db][j] += mg[64 * (16 * db + j)];
      }
    }
    if (ks == 0 && kj < n) {
      float* out = (float*)outp + hoff + (size_t)kj * D;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4)
          Quad<float>::store(out + 32 * db + 8 * q4 + 4 * h, acc[db][4 * q4] * sc, acc[db][4 * q4 + 1] * sc,
                             acc[db][4 * q4 + 2] * sc, acc[db][4 * q4 + 3] * sc);
    }
  };
  finish(dv, a.dv, 1.f);
  finish(dk, a.dk, a.dk_scale);
}

}  // namespace attn
