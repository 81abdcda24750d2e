// Workgroup id -> (head, tile) schedule, on the host and the device (no HIP
// headers needed, so that it can be checked on the CPU).
#pragma once

#ifdef __HIP__
#define ATTN_HD __host__ __device__ __forceinline__
#else
#define ATTN_HD inline
#endif

namespace attn {

constexpr int kXcds = 8, kCusPerXcd = 32;

// Consecutive workgroup ids are dispatched round-robin over the 8 XCDs (each
// with its own L2), in id order within an XCD.
// hgroup == 0 (every tile the same work): each XCD gets a contiguous range of
// (head, tile), so the tiles of one head, which share K and V, run on the
// same L2.
// hgroup > 0 (causal; `reverse`: the last tile of a head has the most work,
// else the first): the heads are taken in groups of hgroup and a group is
// issued tile by tile, from the most work to the least, all its heads at each
// tile; with hgroup a multiple of 8, head i of a group stays on one XCD. An
// XCD then ends on its shortest tiles. Head by head it ended on the longest
// tiles of its last head, started when only a part of the workgroups was
// still running. Measured at n = 4096, 32 heads, d = 128, causal, head by
// head / in groups: forward 196 / 160 us, dK/dV 326 / 265, dQ 245 / 197; at
// n = 16384, 64 heads (groups of 8, one head per XCD) the same to 0.7 %.
// Heads left over (heads mod hgroup) go first, spread over the XCDs.
ATTN_HD void block_map(int bid, int nblocks, int ntiles, int hgroup, bool reverse, int& head, int& tile) {
  int t;
  if (hgroup == 0) {
    const int per = (int)((unsigned)nblocks / kXcds);
    int lin = bid;
    if (bid < per * kXcds) lin = (bid & (kXcds - 1)) * per + (int)((unsigned)bid / kXcds);
    head = (int)((unsigned)lin / (unsigned)ntiles);
    t = lin - head * ntiles;
  } else {
    const int rem = (int)((unsigned)nblocks / (unsigned)ntiles % (unsigned)hgroup), first = rem * ntiles;
    int h0 = 0, g = rem, i = bid;
    if (bid >= first) {
      const int k = (int)((unsigned)(bid - first) / (unsigned)(hgroup * ntiles));
      h0 = rem + k * hgroup;
      g = hgroup;
      i = bid - first - k * hgroup * ntiles;
    }
    t = (int)((unsigned)i / (unsigned)g);
    head = h0 + i - t * g;
  }
  tile = reverse ? ntiles - 1 - t : t;
}

// Heads per group of the causal order, for kernels of which a compute unit
// holds `per_cu` workgroups: enough that a group fills an XCD at least twice
// over, so that the last group ends evenly (list-scheduling model: within
// 1.02-1.07 of the balanced time, single heads 1.24-1.6), and no more, so that
// many workgroups of a head run together and share K and V through L2 (groups
// of 64 heads at n = 16384, d = 128: forward and dK/dV 4 % slower).
ATTN_HD int head_group(int heads, int ntiles, int per_cu) {
  const int want = 2 * kCusPerXcd * per_cu;   // workgroups per XCD and group
  const int g = kXcds * ((want + ntiles - 1) / ntiles);
  return g < heads ? g : heads;
}

// The largest call, in 128-row tiles over all heads, that the kernels for small
// grids (split.hpp) take: up to there they are faster, their quarter-length
// chains of steps outweighing that each key tile serves 32 queries instead of
// 128 or 256. Under the causal mask that holds for about twice the tiles, half
// of them being short. Time of the large-grid kernels over theirs, at the
// last grid within the limit and the first beyond it (tiles: n = 512 / 2048; the
// float32 kernels of both sides have changed since, the split ones becoming up to
// 25 % faster, so that some of their limits lie early):
//   bf16 forward    d=32   192: 1.19 / 1.45, 208: 1.01 / 1.20 |  384: 1.02 / 1.35, 416: 0.95 / 1.36
//   bf16 forward    d=64   128: 1.20 / 1.38, 144: 0.91 / 0.98 |  192: 1.09 / 1.40, 208: 0.99 / 1.33
//   bf16 forward    d=128  128: 1.31 / 1.20, 144: 0.97 / 0.84 |  256: 1.00 / 1.07, 288: 0.93 / 0.98
//   bf16 dK/dV      d=32   192: 1.07 / 1.21, 208: 0.91 / 1.01 |  320: 1.10 / 1.38, 352: 1.07 / 1.36
//   bf16 dK/dV      d=64   256: 1.03 / 1.23, 288: 0.89 / 1.00 |  384: 1.08 / 1.49, 416: 0.97 / 1.32
//   bf16 dK/dV      d=128  112: 0.99 / 1.17, 128: 0.98 / 1.17 |  160: 0.92 / 1.28, 176: 0.87 / 1.13
//   bf16 dQ         d=32   384: 1.06 / 1.16, 416: 0.96 / 1.07 |  384: 1.25 / 1.63, 416: 1.18 / 1.58
//   bf16 dQ         d=64   192: 0.96 / 1.07, 208: 0.81 / 0.86 |  224: 1.06 / 1.60, 256: 0.99 / 1.37
//   bf16 dQ         d=128  128: 1.10 / 1.29, 144: 0.85 / 0.91 |  192: 0.94 / 1.30, 208: 0.88 / 1.21
//   f32  forward    d=32   128: 1.38 / 1.46, 144: 1.01 / 1.02 |  176: 1.26 / 1.54, 192: 1.25 / 1.47
//   f32  forward    d=64   80: 1.24 / 1.29, 96: 1.23 / 1.28 |  128: 1.54 / 1.69, 144: 1.32 / 1.46
//   f32  forward    d=128  128: 1.35 / 1.43, 144: 0.96 / 1.04 |  256: 1.11 / 1.31, 288: 1.00 / 1.25
//   f32  dK/dV      d=32   80: 1.17 / 1.22, 96: 1.16 / 1.21 |  176: 1.07 / 1.44, 192: 0.99 / 1.42
//   f32  dK/dV      d=64   80: 1.06 / 1.06, 96: 1.05 / 1.06 |  192: 0.95 / 1.13, 208: 0.86 / 1.10
//   f32  dK/dV      d=128  80: 1.05 / 1.07, 96: 1.05 / 1.08 |  160: 1.09 / 1.18, 176: 0.79 / 0.84
//   f32  dQ         d=32   80: 1.15 / 1.17, 96: 1.15 / 1.16 |  144: 1.17 / 1.33, 160: 1.12 / 1.24
//   f32  dQ         d=64   80: 1.02 / 0.98, 96: 1.01 / 0.98 |  112: 1.33 / 1.37, 128: 1.34 / 1.32
//   f32  dQ         d=128  128: 1.12 / 1.23, 144: 0.77 / 0.83 |  208: 0.89 / 1.18, 224: 0.91 / 1.18
// With n below 512 a causal head has too few short tiles for the causal limit
// (250 heads, n = 100, bf16, d = 64: 0.91), and at n <= 128 a bf16 backward at
// d = 128 has at most four steps to share (n = 33 to 100, dK/dV: 0.81-0.92).
enum Kind { kFwd, kDkdv, kDq };
constexpr int split_limit(Kind kind, bool b16, int d, bool causal) {
  constexpr int limit[2][3][3][2] = {   // [bf16][kind][d = 32, 64, 128][causal]
      {{{128, 176}, {80, 128}, {128, 256}},
       {{80, 176}, {80, 192}, {80, 160}},
       {{80, 144}, {80, 112}, {128, 208}}},
      {{{192, 384}, {128, 192}, {128, 256}},
       {{192, 320}, {256, 384}, {112, 160}},
       {{384, 384}, {192, 224}, {128, 192}}}};
  return limit[b16][kind][d == 32 ? 0 : d == 64 ? 1 : 2][causal];
}
// The split kernels of the backward run in one launch (bwd_split_kernel) where
// that is faster than two, and than the large-grid kernels: neither fills the
// chip, so they run side by side, and a launch's fixed time is saved (1.4-1.7 up
// to 32 tiles). Time of the better of two split and two large-grid launches over
// one, as above; bf16 at d = 128 and float32 at d >= 64 hold one workgroup per
// compute unit (LDS, registers), which ends them at about half the others' limit:
//   bf16 one launch d=32   320: 1.16 / 1.12, 352: 1.16 / 1.14 |  384: 1.17 / 1.07, 416: 1.17 / 1.03
//   bf16 one launch d=64   256: 1.02 / 1.06, 288: 1.02 / 1.13 |  352: 1.07 / 1.04, 384: 1.02 / 1.01
//   bf16 one launch d=128  112: 1.00 / 1.00, 128: 1.00 / 1.00 |  128: 1.05 / 1.10, 144: 1.10 / 1.08
//   f32  one launch d=32   96: 1.10 / 1.08, 112: 1.06 / 1.01 |  192: 1.17 / 1.08, 208: 1.09 / 1.07
//   f32  one launch d=64   96: 1.28 / 1.29, 112: 1.02 / 1.02 |  176: 1.06 / 1.04, 192: 0.99 / 1.06
//   f32  one launch d=128  96: 1.26 / 1.25, 112: 1.01 / 1.01 |  112: 1.08 / 0.99, 128: 1.02 / 1.01
inline bool one_backward(bool b16, int d, bool causal, int heads, int n) {
  constexpr int limit[2][3][2] = {   // [bf16][d = 32, 64, 128][causal]
      {{104, 192}, {104, 176}, {104, 112}}, {{320, 384}, {256, 352}, {112, 128}}};
  return (long long)heads * ((n + 127) / 128) <= limit[b16][d == 32 ? 0 : d == 64 ? 1 : 2][causal && n >= 512];
}
// (the backward kernels follow one_backward also where they are launched apart,
// so that results do not depend on that)
inline bool use_split(Kind kind, bool b16, int d, bool causal, int heads, int n) {
  if (kind != kFwd && one_backward(b16, d, causal, heads, n)) return true;
  if (b16 && d == 128 && kind != kFwd && n <= 128) return false;
  return (long long)heads * ((n + 127) / 128) <= split_limit(kind, b16, d, causal && n >= 512);
}

// The atomic-dQ form adds a float32 dQ per key block, four times as many from
// 32-key blocks as from 128-key ones, so its dK/dV leaves the split kernel much
// earlier (below the fused path's limits, so that dK and dV are the same bits
// there). Time of the whole call with the split / with the large-grid dK/dV, over
// its time on large-grid kernels throughout, n = 512, 2048, 8192: d = 32 48 tiles 0.94, 0.76 / 1.00, 0.82,
// 64 tiles 0.95, 0.91, 0.92 / 1.01, 0.82, 0.80; d = 64 32 tiles 0.79, 0.71 / 0.87,
// 0.83, 48 tiles 0.95, 0.94 / 0.87, 0.82, 256 tiles 2.5, 3.0, 3.1 / 1.00; d = 128 32
// tiles 0.77, 0.82 / 0.78, 0.83, 48 tiles 0.98, 1.11 / 0.78, 0.83. Causal: d = 32 96
// tiles 0.96, 0.81 / 1.02, 0.82, 128 tiles 1.01, 0.94, 0.92 / 0.97, 0.82, 0.79; d = 64
// 64 tiles 0.86, 0.77, 0.77 / 0.87, 0.82, 0.82, 80 tiles 0.97, 0.95 / 0.89, 0.85; d =
// 128 48 tiles 0.72, 0.73 / 0.79, 0.82, 64 tiles 0.82, 0.85, 0.89 / 0.79, 0.82, 0.84.
inline bool use_split_atomic(int d, bool causal, int heads, int n) {
  constexpr int limit[3][2] = {{48, 96}, {32, 64}, {32, 48}};   // [d = 32, 64, 128][causal]
  return (long long)heads * ((n + 127) / 128) <= limit[d == 32 ? 0 : d == 64 ? 1 : 2][causal && n >= 512];
}

// The float32 kernels of f32x3.hpp come with four waves, or (d <= 64) with
// eight that share every tile. Eight keep two waves on each SIMD while there
// is one workgroup per compute unit; with more, two workgroups of four are
// better, their barriers being independent. Time of eight over four at n = 512
// / 2048, d = 64: 256 tiles forward 0.94 / 0.89, dK/dV 0.84 / 0.80, dQ 0.92 /
// 0.88; 320 tiles 1.14 / 1.08, 1.13 / 1.10, 1.16 / 1.10; causal 384 tiles 1.01 /
// 0.83, 0.84 / 0.72, 0.98 / 0.79, 512 tiles 1.09 / 0.89, 0.95 / 0.79, 1.07 /
// 0.85; d = 32 forward 256 tiles 0.88 / 0.83, 288 tiles 1.11 / 1.05, at n = 128 1.01 and
// 1.30 (1500 heads 1.50), causal 384 tiles 0.97 / 0.77, 416 tiles 1.09 / 0.77.
// (n <= 64 leaves the second four nothing.)
inline bool x3_eight_waves(int d, bool causal, int heads, int n) {
  if (d == 128 || n <= 64) return false;
  return (long long)heads * ((n + 127) / 128) <= (causal && n >= 512 ? 384 : 256);
}

// Tiles per head, grid size and issue order of `heads` heads in tiles of
// `rows` rows (Args: FwdArgs or BwdArgs).
template <typename Args> inline void set_grid(Args& a, int heads, int rows, int per_cu) {
  a.ntiles = (a.n + rows - 1) / rows;
  a.nblocks = heads * a.ntiles;
  a.hgroup = head_group(heads, a.ntiles, per_cu);
}

}  // namespace attn
