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
// of them being short. Time of the large-grid kernels over theirs, measured
// at n = 512 / 2048 / 8192:
//   bf16, d = 128, forward  64 tiles 2.05 / 2.07 / 2.01, 128 tiles 1.38 / 1.18 / 1.10, 192 tiles 1.06 / 0.87 / 0.78
//   the same causal         64 tiles 2.15 / 2.13 / 2.18, 256 tiles 1.11 / 1.11 / 1.05, 384 tiles 0.87 / 0.84 / 0.77
//   bf16, d = 64, dK/dV     64 tiles 2.12 / 2.92 / 3.38, 256 tiles 1.04 / 1.18 / 1.23, 512 tiles 0.83 / 0.81 / 0.81
//   f32, d = 64, dQ         64 tiles 1.54 / 1.65 / 1.68,  96 tiles 0.80 / 0.78,        256 tiles 0.51 / 0.48 / 0.46
//   the same causal         64 tiles 1.57 / 1.69 / 1.71, 128 tiles 0.99 / 0.98 / 1.00, 256 tiles 0.69 / 0.68 / 0.68
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
// chip, so they run side by side, and a launch's fixed time is saved. Time of
// two launches over one: 1.4-1.7 up to 32 tiles; bf16, d = 64, n = 512 / 2048 /
// 8192: 64 tiles 1.32 / 1.29 / 1.31, 256 tiles 1.02 / 1.02 / 1.02, causal 256
// tiles 1.12 / 1.29 / 1.42, 384 tiles 0.99 / 1.09; d = 128 (dK/dV takes a
// compute unit's LDS) 96 tiles 1.24 / 1.25, 128 tiles 0.98 / 1.09 / 1.14, 192
// tiles 0.73 / 0.83; float32, d = 64: 96 tiles 1.20 / 1.20, 128 tiles 0.95 /
// 0.94 / 0.93.
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
// there). Whole call, split / large-grid kernel, in time of the large-grid
// kernels throughout, n = 512 / 2048 / 8192: d = 32 48 tiles 0.94, 0.76 / 1.00, 0.82,
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
