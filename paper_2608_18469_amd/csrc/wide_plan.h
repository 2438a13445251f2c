// When a GEMM runs in the 256x256 tiles of wide.hip (bf16), and how many
// slices its weight gradient's contraction takes: modelled times, from
// measurements on one MI355X (256 compute units).
#pragma once

#include <algorithm>
#include <cstdint>

namespace erase {

// Modelled microseconds of one 256x256 tile of `ks` 64-wide k-steps: the
// phases and the tile's start and epilogue.  Measured, launches of whole
// rounds of 256 workgroups: 16384 x 1024 x 1677 (27 k-steps, one round)
// 50.4 us, 16384 x 2048 x 512 (8 k-steps, two rounds) 41.7 us,
// 8192 x 8192 x 8192 (128 k-steps, four rounds) 930 us.
inline double wide_tile_us(int64_t ks) { return 1.6 * double(ks) + 6.0; }
inline int64_t wide_tiles(int64_t M, int64_t N) { return (M + 255) / 256 * ((N + 255) / 256); }
// Partial slices written by the GEMM and read by Adam, fp32, at 5 TB/s.
inline double wide_part_us(int64_t M, int64_t N, int64_t split) { return 8.0 * double(M) * double(N) * double(split) / 5e6; }
constexpr int kWideCus = 256, kWideMaxSplit = 16;

// Time of n1 jobs of t1 and n2 of t2 handed in order of length to 256 units:
// the long ones fill whole rounds and leave the units on two levels; the
// least time at which the short ones fit on top, by bisection.
inline double wide_makespan(int64_t n1, double t1, int64_t n2, double t2) {
  if (n1 == 0 || (n2 > 0 && t1 < t2)) {
    std::swap(n1, n2);
    std::swap(t1, t2);
  }
  const double full = double(n1 / kWideCus) * t1;
  const int64_t rem = n1 % kWideCus;
  double lo = rem ? full + t1 : full;
  if (n2 == 0) return lo;
  auto room = [&](double T) {
    const double a = T - full - t1, b = T - full;
    return (a > 0 ? rem * int64_t(a / t2) : 0) + (b > 0 ? (kWideCus - rem) * int64_t(b / t2) : 0);
  };
  double hi = lo + t2 * (double(n2) / kWideCus + 2.0);
  if (room(lo) >= n2) return lo;
  for (int i = 0; i < 24; ++i) {
    const double mid = 0.5 * (lo + hi);
    (room(mid) >= n2 ? hi : lo) = mid;
  }
  return hi;
}

// Forward and input-gradient GEMMs [M][N] over K: wide tiles when they beat
// the 128x128 tiles of the GEMM core (two workgroups per compute unit).
// Measured 128x128 against 256x256: 16384 x 1677 x 1677 138 and 94 us,
// 16384 x 512 x 1024 30.4 and 30.9 us, 4096 x 512 x 1677 25.7 and 38.7 us.
inline bool wide_nt_pays(int64_t M, int64_t N, int64_t K) {
  const int64_t ks = (K + 63) / 64, t = wide_tiles(M, N);
  const int64_t t128 = (M + 127) / 128 * ((N + 127) / 128);
  if (t < 128) return false;
  const double wide = double((t + kWideCus - 1) / kWideCus) * wide_tile_us(ks);
  const double core = double((t128 + 511) / 512) * (1.28 * double(ks) + 6.0);
  return wide < core;
}

struct WideSplit {
  int split = 0;  // 0: nothing below the limit
  double us = 0;  // GEMM, and the partial slices' traffic
};
// Weight gradient [M][N] over K batch rows, alone (nd = 0) or in one launch
// with nd input-gradient tiles of kd k-steps: the slice count of the
// shortest modelled time below `limit`.
inline WideSplit wide_wgrad_split(int64_t M, int64_t N, int64_t K, double limit, int64_t nd = 0, int64_t kd = 0) {
  const int64_t ks = std::max<int64_t>(1, (K + 63) / 64), nw = wide_tiles(M, N);
  WideSplit best{0, limit};
  for (int s = 1; s <= kWideMaxSplit && (s == 1 || ks / s >= 8); ++s) {
    const double tw = wide_tile_us((ks + s - 1) / s), td = wide_tile_us(kd), part = wide_part_us(M, N, s);
    // least possible: the longest tile, and every unit busy throughout
    if (std::max(std::max(tw, nd ? td : 0.0), (double(nw * s) * tw + double(nd) * td) / kWideCus) + part >= best.us) continue;
    const double us = wide_makespan(nw * s, tw, nd, td) + part;
    if (us < best.us) best = {s, us};
  }
  return best;
}

// A layer's two backward GEMMs (weight gradient [Nout][Kin] over M rows, input
// gradient [M][Kin] over Nout): the slices of the weight gradient when the
// wide launch beats the core's grouped 64x64 one (420 TFLOP/s on the large
// shapes: 2 x 16384 x 1024 x 1677 in 273-395 us), else 0.
inline int wide_pair_split(int64_t M, int64_t Nout, int64_t Kin) {
  const double core = 4.0 * double(M) * double(Nout) * double(Kin) / 420e6 + 4.0;
  return wide_wgrad_split(Nout, Kin, M, core, wide_tiles(M, Kin), (Nout + 63) / 64).split;
}

// The core's split 64x64 weight gradient alone (512 x 2048 over 16384 rows:
// 75 us).
inline double wide_core_wgrad_us(int64_t M, int64_t N, int64_t K) {
  return 2.0 * double(M) * double(N) * double(K) / 460e6 + 4.0;
}

}  // namespace erase
