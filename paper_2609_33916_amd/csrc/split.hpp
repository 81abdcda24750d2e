// Kernels for grids that leave most of the chip idle: a workgroup owns 32 rows
// (queries in the forward and dQ, keys in dK/dV) and its four waves share the
// streamed dimension, wave w taking the 32-row blocks w, w + 4, w + 8, ... on
// its own; the waves' partial results are merged through LDS once, at the end.
// Against the 128- and 256-row kernels a call has 4 to 8 times the workgroups
// and each has a quarter of the steps, with no barrier in the loop.
//
// These grids are bound by the length of a workgroup's chain of steps (and a
// launch's fixed 5 to 7 us), not by any unit's rate. Measured, large-grid
// kernels / these (us): 16 heads, n = 1000, d = 128, causal, bf16: forward 37 /
// 23, dK/dV 44 / 30, dQ 35 / 24; 1 head, n = 1024, d = 64, bf16: 20 / 11,
// 34 / 13, 23 / 11; 8 heads, n = 1024, d = 64, float32: 81 / 27, 153 / 47,
// 116 / 38. The limits are in grid.hpp.
//
// Operands that are read as rows (contraction over d) go from global memory
// straight into registers as the matrix operand; in bfloat16 the operands read
// transposed go through LDS tiles that belong to one wave (LDS DMA, two
// stages), in float32 they are 4-byte loads, one row of 32 columns per lane
// half, also straight into registers. Rows past the end repeat the last row
// and are masked (the float32 transposed operands read zeros there).
#pragma once

#include "kernels.hpp"

namespace attn {

// Until at most N vector-memory operations (in issue order) are outstanding.
template <int N> __device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt has 6 bits");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));   // expcnt, lgkmcnt: no wait
  asm volatile("" ::: "memory");
}

// Copy of 32 rows of a [n, D] bf16 matrix into a 32-row tile (the permuted,
// swizzled layout of RowRead / TransRead) by one wave. Rows >= n fetch row
// n - 1.
template <int D> struct WaveTile {
  static constexpr int C = D / 8, NI = D / 16;   // chunks per row; 1 KB copies
  static constexpr int ELEMS = 32 * D;
  int off[NI], xr[NI];
  __device__ __forceinline__ explicit WaveTile(int lane) {
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int L = 64 * j + lane, s = L / C, slot = L % C;
      xr[j] = perm32(s);
      off[j] = xr[j] * D + 8 * (slot ^ swz<D>(s));
    }
  }
  __device__ __forceinline__ void issue(bf16* lds, const bf16* g, int row0, int n) const {
    const auto rs = dma_rsrc(g + (size_t)row0 * D);
    const bool full = row0 + 32 <= n;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      int o = off[j];
      if (!full) o -= max(row0 + xr[j] - (n - 1), 0) * D;
      dma16(rs, 2u * (unsigned)o, (ATTN_LDS void*)(lds + 512 * j));
    }
  }
};

// Row operands of one row per lane, as loaded: 16-byte chunks, chunk u of lane
// half h holding the columns of the bf16 k-step u (16u + 8h + [0, 8)), or in
// float32 the k-steps 4u + [0, 4) (columns 8u + 4h + [0, 4)).
template <typename T, int D> struct RowRegs {
  static constexpr int NU = D * sizeof(T) / 32;
  u32x4 r[NU];
  __device__ __forceinline__ void load(const T* row, int h, uint32_t flip = 0u) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      r[u] = *(const u32x4*)(row + (2 * u + h) * Elem<T>::CH);
      r[u] ^= (u32x4){flip, flip, flip, flip};
    }
  }
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int u = 0; u < NU; ++u) r[u] = (u32x4){0u, 0u, 0u, 0u};
  }
};
// acc += A B^T over d, rows of A and of B in registers
template <int D> __device__ __forceinline__ void mma_rows(f32x16& acc, const RowRegs<bf16, D>& a, const RowRegs<bf16, D>& b) {
#pragma unroll
  for (int u = 0; u < RowRegs<bf16, D>::NU; ++u) mma(acc, __builtin_bit_cast(bf16x8, a.r[u]), __builtin_bit_cast(bf16x8, b.r[u]));
}
template <int D> __device__ __forceinline__ void mma_rows(f32x16& acc, const RowRegs<float, D>& a, const RowRegs<float, D>& b) {
#pragma unroll
  for (int u = 0; u < RowRegs<float, D>::NU; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) mma(acc, __uint_as_float(a.r[u][e]), __uint_as_float(b.r[u][e]));
}

// float32: columns of 32 rows as transposed operands (row 16h + t for k-step
// t), loaded R k-steps ahead of their products (a k-step's products take
// 64 D/32 cycles, so 8 steps, or 4 at d = 128, cover a load from L2). Buffer
// loads, whose range ends with the matrix: rows past the end read as zeros (the
// other operand is zero there, and a repeated last row may hold an infinity). The
// whole offset is the vector one, which the range check covers.
template <int D> struct ColRegs {
  static constexpr int NDB = D / 32, R = D == 128 ? 4 : 8;
  float v[R][NDB];
  __amdgpu_buffer_rsrc_t rs;
  unsigned off;   // in bytes
  // x: a [n, D] matrix (below 2 GB: small grids)
  __device__ __forceinline__ ColRegs(const float* x, int n)
      : rs(__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(x), (short)0, n * D * 4, 0x00020000)) {}
  __device__ __forceinline__ void get(int t) {
#pragma unroll
    for (int db = 0; db < NDB; ++db)
      v[t % R][db] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, off + 4u * (t * D + 32 * db), 0, 0));
  }
  // the first R k-steps of rows [r0, r0 + 32)
  __device__ __forceinline__ void load(int r0, int h, int c) {
    off = 4u * (unsigned)((r0 + 16 * h) * D + c);
#pragma unroll
    for (int t = 0; t < R; ++t) get(t);
  }
};
// acc += A^T B over the 32 rows
template <int D>
__device__ __forceinline__ void mma_cols(f32x16 (&acc)[D / 32], ColRegs<D>& a, const f32x16& b) {
#pragma unroll
  for (int t = 0; t < 16; ++t) {
#pragma unroll
    for (int db = 0; db < D / 32; ++db) mma(acc[db], a.v[t % ColRegs<D>::R][db], b[t]);
    if (t + ColRegs<D>::R < 16) a.get(t + ColRegs<D>::R);
  }
}
// bf16: the same from an LDS tile
template <int D> __device__ __forceinline__ void mma_cols(f32x16 (&acc)[D / 32], const bf16* tile, const f32x16& b, int h, int c) {
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const bf16x8 f = FragFromAcc<bf16>::get(b, t);
#pragma unroll
    for (int db = 0; db < D / 32; ++db) mma(acc[db], TransRead<bf16, D, 32>::get(tile, 0, db, t, h, c), f);
  }
}

// ------------------------------------------------------- merging the waves --
// A wave's transposed accumulator (lane (h, c): columns 32db + 8q4 + 4h + [0, 4)
// of row c) in LDS, as [wave][row][chunk of 4 columns]: columns below D/2 in
// lo, the others in hi; a row's chunks are XOR-swizzled by the row.
template <int D> struct WaveMerge {
  static constexpr int NCH = D / 8;                 // chunks per row and half
  static constexpr int FLOATS = 4 * 32 * (D / 2);   // per half
  __device__ __forceinline__ static f32x4* at(float* lo, float* hi, int w, int row, int ch) {
    return (f32x4*)(ch < NCH ? lo : hi) + (w * 32 + row) * NCH + ((ch & (NCH - 1)) ^ (row & (NCH - 1)));
  }
  __device__ __forceinline__ static void put(float* lo, float* hi, int w, int h, int c, const f32x16 (&acc)[D / 32]) {
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        *at(lo, hi, w, c, 8 * db + 2 * q4 + h) =
            (f32x4){acc[db][4 * q4], acc[db][4 * q4 + 1], acc[db][4 * q4 + 2], acc[db][4 * q4 + 3]};
  }
  // chunk `ch` of `row`, the four waves weighted by f
  __device__ __forceinline__ static f32x4 get(float* lo, float* hi, int row, int ch, const float (&f)[4]) {
    f32x4 r = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const f32x4 x = *at(lo, hi, w, row, ch);
#pragma unroll
      for (int e = 0; e < 4; ++e) r[e] = fmaf(f[w], x[e], r[e]);
    }
    return r;
  }
};

// ======================================================================
// Forward. Per wave and 32-key block: S^T = K Q^T (rows = keys, cols = the
// workgroup's 32 queries), online softmax per column, O^T += V^T P^T; the
// waves' (max, sum, O) are merged by log-sum-exp.
// ======================================================================
template <typename T, int D, bool CAUSAL>
__global__ void __launch_bounds__(256, sizeof(T) == 4 && D == 128 ? 1 : 2) fwd_split_kernel(const FwdArgs a) {
  constexpr int NDB = D / 32;
  constexpr bool B16 = sizeof(T) == 2;
  using MG = WaveMerge<D>;
  // V tiles of the four waves, two stages, in distinct LDS objects (the loop
  // is unrolled by two, so that reads of one stage never wait for the copy
  // into the other); afterwards the merge buffers
  __shared__ __attribute__((aligned(16))) float stA[MG::FLOATS];
  __shared__ __attribute__((aligned(16))) float stB[MG::FLOATS];
  __shared__ float ml[2][4][32];

  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, c = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int head, qt;
  block_map(blockIdx.x, a.nblocks, a.ntiles, CAUSAL ? a.hgroup : 0, CAUSAL, head, qt);
  const int n = a.n, q0 = 32 * qt, qi = q0 + c;
  const size_t hoff = (size_t)head * (size_t)a.head_stride;
  const T* Kg = (const T*)a.k + hoff;
  const T* Vg = (const T*)a.v + hoff;
  const int nb = ((CAUSAL ? min(n, q0 + 32) : n) + 31) / 32;   // key blocks
  const float sl2 = a.sl2;

  f32x16 oacc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) oacc[db] = zero16();
  float m_use = -INFINITY, lsum = 0.f;

  RowRegs<T, D> q;
  // S of key block kb -> P, moving the running maximum and sum
  auto softmax = [&](int kb, f32x16& s) __attribute__((always_inline)) {
    const int kv0 = 32 * kb;
    if (kv0 + 32 > n || (CAUSAL && kv0 + 31 > q0)) {
      const int lim = (CAUSAL ? min(qi, n - 1) : n - 1) - (kv0 + 16 * h);
#pragma unroll
      for (int j = 0; j < 16; ++j) s[j] = (j > lim) ? -INFINITY : s[j];
    }
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < 16; ++j) mx = fmaxf(mx, s[j]);
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
    float rs = 0.f;   // a block's sum first: thousands of single terms would lose bits in lsum
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      s[j] = exp2_fast(fmaf(s[j], sl2, mb));
      rs += s[j];
    }
    lsum += rs;
  };
  // the K rows of a block in accumulator order: lane c takes key perm32(c)
  auto kload = [&](int kb, RowRegs<T, D>& k) __attribute__((always_inline)) {
    k.load(Kg + (size_t)min(32 * kb + perm32(c), n - 1) * D, h);
  };

  if constexpr (B16) {
    const WaveTile<D> vt(lane);
    bf16* const vA = (bf16*)stA + w * WaveTile<D>::ELEMS;
    bf16* const vB = (bf16*)stB + w * WaveTile<D>::ELEMS;
    RowRegs<T, D> kA, kB;
    if (w < nb) {
      vt.issue(vA, Vg, 32 * w, n);
      kload(w, kA);
    }
    if (qi < n) q.load((const T*)a.q + hoff + (size_t)qi * D, h, a.qflip);
    else q.zero();
    auto step = [&](int kb, bf16* vc, RowRegs<T, D>& kc, bf16* vn, RowRegs<T, D>& kn) __attribute__((always_inline)) {
      if (kb + 4 < nb) {
        vt.issue(vn, Vg, 32 * (kb + 4), n);
        kload(kb + 4, kn);
        wait_vm<WaveTile<D>::NI + RowRegs<T, D>::NU>();   // this block's V and K are there
      } else {
        wait_vm<0>();
      }
      f32x16 s = zero16();
      mma_rows<D>(s, kc, q);
      softmax(kb, s);
      mma_cols<D>(oacc, vc, s, h, c);
      __builtin_amdgcn_s_waitcnt(0xC07F);   // V reads done (lgkmcnt 0) before the stage is refilled
    };
    for (int kb = w; kb < nb; kb += 8) {
      step(kb, vA, kA, vB, kB);
      if (kb + 4 < nb) step(kb + 4, vB, kB, vA, kA);
    }
  } else {
    RowRegs<T, D> k;
    ColRegs<D> v(Vg, n);
    if (w < nb) {
      kload(w, k);
      v.load(32 * w, h, c);
    }
    if (qi < n) q.load((const T*)a.q + hoff + (size_t)qi * D, h, a.qflip);
    else q.zero();
    for (int kb = w; kb < nb; kb += 4) {
      f32x16 s = zero16();
      mma_rows<D>(s, k, q);
      if (kb + 4 < nb) kload(kb + 4, k);
      softmax(kb, s);
      mma_cols<D>(oacc, v, s);
      if (kb + 4 < nb) v.load(32 * (kb + 4), h, c);
    }
  }

  // ---- merge: thread -> query qq and the 4-column chunks dp + 8e
  const float lw = halves_sum(lsum);
  __syncthreads();
  if (h == 0) {
    ml[0][w][c] = m_use;
    ml[1][w][c] = lw;
  }
  MG::put(stA, stB, w, h, c, oacc);
  __syncthreads();
  const int qq = tid >> 3, dp = tid & 7, qr = q0 + qq;
  float M = -INFINITY, f[4], l = 0.f;
#pragma unroll
  for (int v = 0; v < 4; ++v) M = fmaxf(M, ml[0][v][qq]);
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    f[v] = (M == -INFINITY) ? 0.f : exp2_fast(ml[0][v][qq] - M);   // -inf: a wave without keys, or scores of -inf
    l += f[v] * ml[1][v][qq];
  }
  const float inv = 1.f / l;
#pragma unroll
  for (int v = 0; v < 4; ++v) f[v] *= inv;
  float dsum = 0.f;
  if (qr < n) {
    const size_t ro = hoff + (size_t)qr * D;
    f32x4 g[NDB];
    if (a.dout) {
#pragma unroll
      for (int e = 0; e < NDB; ++e) g[e] = Quad<T>::load((const T*)a.dout + ro + 4 * (dp + 8 * e));
    }
#pragma unroll
    for (int e = 0; e < NDB; ++e) {
      const f32x4 o = MG::get(stA, stB, qq, dp + 8 * e, f);
      Quad<T>::store((T*)a.o + ro + 4 * (dp + 8 * e), o[0], o[1], o[2], o[3]);
      if (a.dout) dsum += o[0] * g[e][0] + o[1] * g[e][1] + o[2] * g[e][2] + o[3] * g[e][3];
    }
  }
#pragma unroll
  for (int x = 1; x < 8; x <<= 1) dsum += __shfl_xor(dsum, x);
  if (qr < n && dp == 0) {
    const size_t row = (size_t)head * n + qr;
    const float l2 = M + log2f(l);
    a.lse[row] = l2 * kLn2;
    if (a.dout) {
      a.dvec[row] = -dsum;   // stored negated (the backward starts dP - D from it)
      a.lse2[row] = l2;
    }
  }
}

// ======================================================================
// dQ. Per wave and 32-key block: S^T = K Q^T, dP^T = V dO^T, dS^T =
// P^T (dP^T - D), dQ^T += K^T dS^T; the waves' dQ are added.
// ======================================================================
template <typename T, int D, bool CAUSAL>
__device__ __forceinline__ void dq_split(const BwdArgs& a, int bid, float* stA, float* stB) {
  constexpr int NDB = D / 32;
  constexpr bool B16 = sizeof(T) == 2;
  using MG = WaveMerge<D>;

  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, c = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int head, qt;
  block_map(bid, a.nblocks, a.ntiles, CAUSAL ? a.hgroup : 0, CAUSAL, head, qt);
  const int n = a.n, q0 = 32 * qt, qi = q0 + c;
  const size_t hoff = (size_t)head * (size_t)a.head_stride;
  const T* Kg = (const T*)a.k + hoff;
  const T* Vg = (const T*)a.v + hoff;
  const int nb = ((CAUSAL ? min(n, q0 + 32) : n) + 31) / 32;
  const float sl2 = a.sl2;

  f32x16 dqa[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) dqa[db] = zero16();
  RowRegs<T, D> q, g;
  float lq = 0.f, nd = 0.f;   // base-2 log-sum-exp and -D of this lane's query
  auto own = [&]() __attribute__((always_inline)) {
    if (qi < n) {
      q.load((const T*)a.q + hoff + (size_t)qi * D, h, a.qflip);
      g.load((const T*)a.dout + hoff + (size_t)qi * D, h);
      lq = a.lse2[(size_t)head * n + qi];
      nd = a.dvec[(size_t)head * n + qi];
    } else {
      q.zero();
      g.zero();
    }
  };
  // dS of key block kb from S and dP (which becomes dS)
  auto grad = [&](int kb, const f32x16& s, f32x16& dp) __attribute__((always_inline)) {
    const int kv0 = 32 * kb;
    const bool edge = kv0 + 32 > n || (CAUSAL && kv0 + 31 > q0);
    const int lim = (CAUSAL ? min(qi, n - 1) : n - 1) - (kv0 + 16 * h);
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      float p = exp2_fast(fmaf(s[j], sl2, -lq));
      if (edge) p = (j > lim) ? 0.f : p;
      dp[j] = p * (dp[j] + nd);
    }
  };
  auto rows = [&](const T* x, int kb, RowRegs<T, D>& r) __attribute__((always_inline)) {
    r.load(x + (size_t)min(32 * kb + perm32(c), n - 1) * D, h);
  };

  if constexpr (B16) {
    const WaveTile<D> kt(lane);
    bf16* const tA = (bf16*)stA + w * WaveTile<D>::ELEMS;
    bf16* const tB = (bf16*)stB + w * WaveTile<D>::ELEMS;
    RowRegs<T, D> v;
    if (w < nb) {
      kt.issue(tA, Kg, 32 * w, n);
      rows(Vg, w, v);
    }
    own();
    auto step = [&](int kb, bf16* tc, bf16* tn) __attribute__((always_inline)) {
      wait_vm<0>();   // this block's K tile and V rows
      if (kb + 4 < nb) kt.issue(tn, Kg, 32 * (kb + 4), n);
      f32x16 dp = zero16(), s = zero16();
      mma_rows<D>(dp, v, g);
      if (kb + 4 < nb) rows(Vg, kb + 4, v);
#pragma unroll
      for (int t = 0; t < D / 16; ++t) mma(s, RowRead<bf16, D>::get(tc, 0, t, h, c), __builtin_bit_cast(bf16x8, q.r[t]));
      grad(kb, s, dp);
      mma_cols<D>(dqa, tc, dp, h, c);
      __builtin_amdgcn_s_waitcnt(0xC07F);
    };
    for (int kb = w; kb < nb; kb += 8) {
      step(kb, tA, tB);
      if (kb + 4 < nb) step(kb + 4, tB, tA);
    }
  } else {
    RowRegs<T, D> k, v;
    ColRegs<D> kc(Kg, n);
    if (w < nb) {
      rows(Kg, w, k);
      rows(Vg, w, v);
      kc.load(32 * w, h, c);
    }
    own();
    for (int kb = w; kb < nb; kb += 4) {
      const bool more = kb + 4 < nb;
      f32x16 s = zero16(), dp = zero16();
      mma_rows<D>(s, k, q);
      if (more) rows(Kg, kb + 4, k);
      mma_rows<D>(dp, v, g);
      if (more) rows(Vg, kb + 4, v);
      grad(kb, s, dp);
      mma_cols<D>(dqa, kc, dp);
      if (more) kc.load(32 * (kb + 4), h, c);
    }
  }

  __syncthreads();
  MG::put(stA, stB, w, h, c, dqa);
  __syncthreads();
  const int qq = tid >> 3, dp = tid & 7, qr = q0 + qq;
  if (qr < n) {
    const float sc = a.dq_scale, f[4] = {sc, sc, sc, sc};
#pragma unroll
    for (int e = 0; e < NDB; ++e) {
      const f32x4 o = MG::get(stA, stB, qq, dp + 8 * e, f);
      Quad<T>::store((T*)a.dq + hoff + (size_t)qr * D + 4 * (dp + 8 * e), o[0], o[1], o[2], o[3]);
    }
  }
}

// ======================================================================
// dK, dV. The workgroup owns 32 keys; per wave and 32-query block:
// S = Q K^T, dP = dO V^T (rows = queries, cols = the keys), P, dS,
// dV^T += dO^T P, dK^T += Q^T dS; the waves' dK and dV are added, dV first
// (one merge buffer).
// With AQ (bf16, the atomic-dQ form; dK and dV are the same bits) a wave also
// passes its dS through an LDS tile [keys][queries] to form dQ = dS K of the
// block, added to the float32 accumulator with atomic adds.
// ======================================================================
template <typename T, int D, bool AQ> struct DkdvLds {
  // bf16: Q tiles, then dO tiles of the four waves, per stage
  static constexpr int STF = WaveMerge<D>::FLOATS * (sizeof(T) == 2 ? 2 : 1);
  static constexpr int KBL = AQ ? 32 * D : 8;     // AQ: the workgroup's K rows
  static constexpr int DST = AQ ? 32 * 32 : 8;    // AQ: each wave's dS^T
};
template <typename T, int D, bool CAUSAL, bool AQ>
__device__ __forceinline__ void dkdv_split(const BwdArgs& a, int bid, float* stA, float* stB, float (&ldA)[4][2][64],
                                           float (&ldB)[4][2][64], bf16* kbl, bf16 (*dst)[DkdvLds<T, D, AQ>::DST]) {
  static_assert(!AQ || sizeof(T) == 2, "the atomic-dQ form is bf16");
  constexpr int NDB = D / 32;
  constexpr bool B16 = sizeof(T) == 2;
  using MG = WaveMerge<D>;

  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, c = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int head, kt;
  block_map(bid, a.nblocks, a.ntiles, CAUSAL ? a.hgroup : 0, false, head, kt);
  const int n = a.n, k0 = 32 * kt, kj = k0 + c;
  const size_t hoff = (size_t)head * (size_t)a.head_stride;
  const T* Qg = (const T*)a.q + hoff;
  const T* dOg = (const T*)a.dout + hoff;
  const auto Lr = dma_rsrc(a.lse2 + (size_t)head * n);
  const auto Dr = dma_rsrc(a.dvec + (size_t)head * n);
  const int b0 = CAUSAL ? kt : 0, nb = (n + 31) / 32;   // query blocks [b0, nb)
  const float sl2 = a.sl2;

  f32x16 dk[NDB], dv[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) { dk[db] = zero16(); dv[db] = zero16(); }
  // K is read sign-flipped for a negative scale (S = |s| Q (-K)^T)
  RowRegs<T, D> k, v;
  auto own = [&]() __attribute__((always_inline)) {
    if (kj < n) {
      k.load((const T*)a.k + hoff + (size_t)kj * D, h, a.qflip);
      v.load((const T*)a.v + hoff + (size_t)kj * D, h);
    } else {
      k.zero();
      v.zero();
    }
  };
  auto ldrows = [&](int qb, float (&ld)[4][2][64]) __attribute__((always_inline)) {
    const unsigned off = 4u * (unsigned)min(32 * qb + c, n - 1);
    dma4(Lr, off, (ATTN_LDS void*)ld[w][0]);
    dma4(Dr, off, (ATTN_LDS void*)ld[w][1]);
  };
  // P (in s) and dS (in dp) of query block qb; lane (h, c): query 16h + j, key kj
  auto grad = [&](int qb, const float (&ld)[4][2][64], f32x16& s, f32x16& dp) __attribute__((always_inline)) {
    const int qbase = 32 * qb + 16 * h;
    const bool edge = 32 * qb + 32 > n || (CAUSAL && 32 * qb < k0 + 31) || (AQ && k0 + 32 > n);
    const int lo = CAUSAL ? kj - qbase : -1, hi = AQ && kj >= n ? -1 : n - 1 - qbase;
#pragma unroll
    for (int j4 = 0; j4 < 4; ++j4) {
      const f32x4 l4 = *(const f32x4*)&ld[w][0][16 * h + 4 * j4];
      const f32x4 d4 = *(const f32x4*)&ld[w][1][16 * h + 4 * j4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = 4 * j4 + e;
        float p = exp2_fast(fmaf(s[j], sl2, -l4[e]));
        if (edge) p = (j < lo || j > hi) ? 0.f : p;
        s[j] = p;
        dp[j] = p * (dp[j] + d4[e]);   // d4 holds -D
      }
    }
  };

  if constexpr (B16) {
    using WT = WaveTile<D>;
    const WT wt(lane);
    bf16* const tA = (bf16*)stA + w * 2 * WT::ELEMS;
    bf16* const tB = (bf16*)stB + w * 2 * WT::ELEMS;
    auto issue = [&](int qb, bf16* t, float (&ld)[4][2][64]) __attribute__((always_inline)) {
      wt.issue(t, Qg, 32 * qb, n);
      wt.issue(t + WT::ELEMS, dOg, 32 * qb, n);
      ldrows(qb, ld);
    };
    if constexpr (AQ) {
      if (w == 0) wt.issue(kbl, (const bf16*)a.k + hoff, k0, n);
      __syncthreads();
    }
    if (b0 + w < nb) issue(b0 + w, tA, ldA);
    own();
    auto add_dq = [&](int qb, const f32x16& ds) __attribute__((always_inline)) {
      if constexpr (AQ) {
        const int row = srow(c);   // of key c; the lane's queries are 16h + [0, 16)
#pragma unroll
        for (int i = 0; i < 2; ++i)
          *(bf16x8*)(dst[w] + row * 32 + 8 * ((2 * h + i) ^ swz<32>(row))) = FragFromAcc<bf16>::get(ds, i);
        const bf16x8 f0 = TransRead<bf16, 32, 32>::get(dst[w], 0, 0, 0, h, c);
        const bf16x8 f1 = TransRead<bf16, 32, 32>::get(dst[w], 0, 0, 1, h, c);
        float* out = a.dqacc + (size_t)head * n * D + c;
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
          f32x16 acc = zero16();
          mma(acc, f0, TransRead<bf16, D, 32>::get(kbl, 0, db, 0, h, c));
          mma(acc, f1, TransRead<bf16, D, 32>::get(kbl, 0, db, 1, h, c));
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            const int qr = 32 * qb + 8 * (j >> 2) + 4 * h + (j & 3);
            if (qr < n) unsafeAtomicAdd(out + (size_t)qr * D + 32 * db, acc[j]);
          }
        }
      }
    };
    auto step = [&](int qb, bf16* tc, float (&lc)[4][2][64], bf16* tn, float (&ln)[4][2][64])
        __attribute__((always_inline)) {
      if (qb + 4 < nb) {
        issue(qb + 4, tn, ln);
        wait_vm<2 * WT::NI + 2>();
      } else {
        wait_vm<0>();
      }
      f32x16 s = zero16(), dp = zero16();
#pragma unroll
      for (int t = 0; t < D / 16; ++t) {
        mma(s, RowRead<bf16, D>::get(tc, 0, t, h, c), __builtin_bit_cast(bf16x8, k.r[t]));
        mma(dp, RowRead<bf16, D>::get(tc + WT::ELEMS, 0, t, h, c), __builtin_bit_cast(bf16x8, v.r[t]));
      }
      grad(qb, lc, s, dp);
      mma_cols<D>(dv, tc + WT::ELEMS, s, h, c);
      mma_cols<D>(dk, tc, dp, h, c);
      add_dq(qb, dp);
      __builtin_amdgcn_s_waitcnt(0xC07F);
    };
    for (int qb = b0 + w; qb < nb; qb += 8) {
      step(qb, tA, ldA, tB, ldB);
      if (qb + 4 < nb) step(qb + 4, tB, ldB, tA, ldA);
    }
  } else {
    RowRegs<T, D> q, g;
    ColRegs<D> qc(Qg, n), gc(dOg, n);
    auto rows = [&](const T* x, int qb, RowRegs<T, D>& r) __attribute__((always_inline)) {
      r.load(x + (size_t)min(32 * qb + perm32(c), n - 1) * D, h);
    };
    if (b0 + w < nb) {
      rows(Qg, b0 + w, q);
      rows(dOg, b0 + w, g);
      ldrows(b0 + w, ldA);
      gc.load(32 * (b0 + w), h, c);
      qc.load(32 * (b0 + w), h, c);
    }
    own();
    auto step = [&](int qb, float (&lc)[4][2][64], float (&ln)[4][2][64]) __attribute__((always_inline)) {
      const bool more = qb + 4 < nb;
      f32x16 s = zero16(), dp = zero16();
      mma_rows<D>(s, q, k);
      if (more) rows(Qg, qb + 4, q);
      mma_rows<D>(dp, g, v);
      if (more) rows(dOg, qb + 4, g);
      if (more) {
        ldrows(qb + 4, ln);
        wait_vm<2 * RowRegs<T, D>::NU + 2>();   // this block's L and D rows
      } else {
        wait_vm<0>();
      }
      grad(qb, lc, s, dp);
      mma_cols<D>(dv, gc, s);
      if (more) gc.load(32 * (qb + 4), h, c);
      mma_cols<D>(dk, qc, dp);
      if (more) qc.load(32 * (qb + 4), h, c);
      __builtin_amdgcn_s_waitcnt(0xC07F);
    };
    for (int qb = b0 + w; qb < nb; qb += 8) {
      step(qb, ldA, ldB);
      if (qb + 4 < nb) step(qb + 4, ldB, ldA);
    }
  }

  const int kk = tid >> 3, dp8 = tid & 7, kr = k0 + kk;
  auto merge = [&](const f32x16 (&acc)[NDB], void* out, float sc) __attribute__((always_inline)) {
    __syncthreads();
    MG::put(stA, stB, w, h, c, acc);
    __syncthreads();
    if (kr < n) {
      const float f[4] = {sc, sc, sc, sc};
#pragma unroll
      for (int e = 0; e < NDB; ++e) {
        const f32x4 o = MG::get(stA, stB, kk, dp8 + 8 * e, f);
        Quad<T>::store((T*)out + hoff + (size_t)kr * D + 4 * (dp8 + 8 * e), o[0], o[1], o[2], o[3]);
      }
    }
  };
  merge(dv, a.dv, 1.f);
  merge(dk, a.dk, a.dk_scale);
}

// The backward's kernels. bwd_split_kernel runs both in one launch, the dK/dV
// workgroups first.
template <typename T, int D, bool CAUSAL>
__global__ void __launch_bounds__(256, sizeof(T) == 4 && D >= 64 ? 1 : 2) dq_split_kernel(const BwdArgs a) {
  // K tiles in two distinct LDS objects, as V's in the forward
  __shared__ __attribute__((aligned(16))) float stA[WaveMerge<D>::FLOATS];
  __shared__ __attribute__((aligned(16))) float stB[WaveMerge<D>::FLOATS];
  dq_split<T, D, CAUSAL>(a, blockIdx.x, stA, stB);
}
template <typename T, int D, bool CAUSAL, bool AQ>
__global__ void __launch_bounds__(256, sizeof(T) == 4 || D == 128 ? 1 : 2) dkdv_split_kernel(const BwdArgs a) {
  using L = DkdvLds<T, D, AQ>;
  __shared__ __attribute__((aligned(16))) float stA[L::STF];
  __shared__ __attribute__((aligned(16))) float stB[L::STF];
  // base-2 log-sum-exp and -D rows of each wave's block
  __shared__ __attribute__((aligned(16))) float ldA[4][2][64];
  __shared__ __attribute__((aligned(16))) float ldB[4][2][64];
  __shared__ __attribute__((aligned(16))) bf16 kbl[L::KBL];
  __shared__ __attribute__((aligned(16))) bf16 dst[4][L::DST];
  dkdv_split<T, D, CAUSAL, AQ>(a, blockIdx.x, stA, stB, ldA, ldB, kbl, dst);
}
template <typename T, int D, bool CAUSAL>
__global__ void __launch_bounds__(256, sizeof(T) == 4 || D == 128 ? 1 : 2) bwd_split_kernel(const BwdArgs a) {
  using L = DkdvLds<T, D, false>;
  __shared__ __attribute__((aligned(16))) float stA[L::STF];
  __shared__ __attribute__((aligned(16))) float stB[L::STF];
  __shared__ __attribute__((aligned(16))) float ldA[4][2][64];
  __shared__ __attribute__((aligned(16))) float ldB[4][2][64];
  const int bid = blockIdx.x;
  if (bid < a.nblocks) dkdv_split<T, D, CAUSAL, false>(a, bid, stA, stB, ldA, ldB, nullptr, nullptr);
  else dq_split<T, D, CAUSAL>(a, bid - a.nblocks, stA, stB);
}

}  // namespace attn
