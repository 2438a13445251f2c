// Which GEMMs run in the 256x256 and 128x128 tiles of wide.hip (bf16), and how
// many slices a weight gradient's contraction takes: modelled times, from
// measurements on one MI355X (256 compute units).  `share` is the number of
// blocks whose launches go out together.
#pragma once

#include <algorithm>
#include <cstdint>

namespace erase {

// Modelled microseconds of one 256x256 tile of `ks` 64-wide k-steps (one on a
// compute unit): the phases and the tile's start and epilogue.  Measured,
// launches of whole rounds of 256 workgroups: 16384 x 1024 x 1677 (27 k-steps,
// one round) 50.4 us, 16384 x 2048 x 512 (8 k-steps, two rounds) 41.7 us,
// 8192 x 8192 x 8192 (128 k-steps, four rounds) 930 us; weight gradients
// (k-major, twice the LDS reads) 1677 x 1677 over 5 x 3277 rows 112 us, 512 x
// 1677 over 16 x 2048 rows 73 us.
inline double wide_tile_us(int64_t ks) { return 1.55 * double(ks) + 7.0; }
inline double wide_wgrad_us(int64_t ks) { return 2.0 * double(ks) + 7.0; }
// A k-step of a 128x128 tile, with two workgroups on a unit and (alone) with
// one; about 7 us more a launch.  16384 x 512 over 512, 1024, 2048 (512 tiles)
// 14.3, 20.6, 34.1 us; 8192 x 512 x 1677 (256 tiles) 18.3 us; weight gradients
// 2006 x 1003 over 4 x 750 rows (512 tiles) 21.4 us, 512 x 1024 over 8 x 2048
// rows (256 tiles) 26.2 us.
constexpr double kMidNt = 0.87, kMidWgrad = 1.25, kMidNtAlone = 0.45, kMidWgradAlone = 0.6;
inline int64_t mid_tiles(int64_t M, int64_t N) { return (M + 127) / 128 * ((N + 127) / 128); }
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

// Forward and input-gradient GEMMs [M][N] over K: 256, 128 or (smaller tiles
// of the core) 0.  Measured 256x256, 128x128 and the core's best: 16384 x
// 1677 x 1677 92, 101 and 135 us; 24576 x 512 x 1677 45.5, 47.3 and 58; 16384 x
// 512 x 1024 29, 20.6 and 29; 3001 x 1003 x 1003 (192 tiles) 27, 12.1 and 15.8;
// 3001 x 600 x 1003 (120) 25, 11.1 and 11.9; 4096 x 256 x 512 (64) 17, 7.6 and
// 7.0; 1000 x 401 x 1003 (32) 25, 10.5 and 8.4 us.  The core's 64x128 tiles with
// two k-groups, one per compute unit, win on a long contraction: 4096 x
// 512 x 1677 (128 tiles of 128x128) 16.2 against 13.3 us.
inline int wide_nt_tile(int64_t M, int64_t N, int64_t K, int share) {
  const int64_t ks = (K + 63) / 64, t = wide_tiles(M, N) * share, tm = mid_tiles(M, N) * share;
  const bool kg2 = K >= 1024 && (M + 63) / 64 * ((N + 127) / 128) >= kWideCus;
  if (tm < (kg2 ? 144 : 112)) return 0;
  const double rounds = double(tm) / 512;
  const double mid = tm <= kWideCus ? kMidNtAlone * double(ks) + 6.0
                                    : kMidNt * double(ks) * 0.5 * (std::max(1.0, rounds) + double((tm + 511) / 512)) + 8.0;
  const double wide = double((t + kWideCus - 1) / kWideCus) * wide_tile_us(ks);
  return t >= 128 && wide < 1.03 * mid ? 256 : 128;
}

struct WideSplit {
  int split = 0;  // 0: nothing below the limit
  double us = 0;  // GEMM, and the partial slices' traffic
};
// Weight gradient [M][N] over K batch rows, alone (nd = 0) or in one launch
// with nd input-gradient tiles of kd k-steps: the slice count of the
// shortest modelled time below `limit`, in 256x256 tiles.
inline WideSplit wide_wgrad_split(int64_t M, int64_t N, int64_t K, double limit, int share, int64_t nd = 0,
                                  int64_t kd = 0) {
  const int64_t ks = std::max<int64_t>(1, (K + 63) / 64), nw = wide_tiles(M, N) * share;
  WideSplit best{0, limit};
  for (int s = 1; s <= kWideMaxSplit && (s == 1 || ks / s >= 8); ++s) {
    const double tw = wide_wgrad_us((ks + s - 1) / s), td = wide_tile_us(kd), part = wide_part_us(M, N, s * share);
    // least possible: the longest tile, and every unit busy throughout
    if (std::max(std::max(tw, nd ? td : 0.0), (double(nw * s) * tw + double(nd) * td) / kWideCus) + part >= best.us) continue;
    const double us = wide_makespan(nw * s, tw, nd, td) + part;
    if (us < best.us) best = {s, us};
  }
  return best;
}
// The same in 128x128 tiles, two on a unit (tiles wait for each other's
// operands, so a launch takes the sum of the work, at least its longest tile).
inline WideSplit mid_wgrad_split(int64_t M, int64_t N, int64_t K, double limit, int share, int64_t nd = 0,
                                 int64_t kd = 0) {
  const int64_t ks = std::max<int64_t>(1, (K + 63) / 64), nw = mid_tiles(M, N) * share;
  WideSplit best{0, limit};
  for (int s = 1; s <= kWideMaxSplit && (s == 1 || ks / s >= 4); ++s) {
    const int64_t kss = (ks + s - 1) / s, t = nw * s + nd;
    const double work = t <= kWideCus ? 0.0
                                      : (kMidWgrad * double(nw * s * kss) + kMidNt * double(nd * kd) + 2.0 * double(t)) / 512;
    const double longest = std::max(kMidWgradAlone * double(kss), nd ? kMidNtAlone * double(kd) : 0.0);
    const double us = std::max(work, longest) + 7.0 + wide_part_us(M, N, s * share);
    if (us < best.us) best = {s, us};
  }
  return best;
}

struct WidePair {
  int tile = 0, split = 1;  // 0: the core's
};
// Weight gradient [M][N] over K rows; core_us: what it takes otherwise.
inline WidePair wide_wgrad(int64_t M, int64_t N, int64_t K, double core_us, int share) {
  const WideSplit m = mid_wgrad_split(M, N, K, core_us, share);
  const WideSplit w = wide_wgrad_split(M, N, K, m.us, share);
  return w.split ? WidePair{256, w.split} : m.split ? WidePair{128, m.split} : WidePair{};
}
// A layer's two backward GEMMs (weight gradient [Nout][Kin] over M rows, input
// gradient [M][Kin] over Nout) against the core's grouped 64x64 launch: 3001 x
// 1003 x 1003 35 us, x 600 x 1003 24.7, x 600 x 300 11.7 us; 4096 x 512 x 256 9.9
// us; 16384 x 1024 x 1677 273 us and more.
inline WidePair wide_pair(int64_t M, int64_t Nout, int64_t Kin, int share) {
  const double core = 4.0 * double(M) * double(Nout) * double(Kin) * share / 450e6 + 6.0;
  const int64_t kd = (Nout + 63) / 64;
  const WideSplit m = mid_wgrad_split(Nout, Kin, M, core, share, mid_tiles(M, Kin) * share, kd);
  const WideSplit w = wide_wgrad_split(Nout, Kin, M, m.us, share, wide_tiles(M, Kin) * share, kd);
  return w.split ? WidePair{256, w.split} : m.split ? WidePair{128, m.split} : WidePair{};
}
// The vocabulary head's backward pair: weight gradient [V][d] over N positions
// and input gradient [N][d] over the vocabulary, whose few tiles are each a long
// chain (1800 x 192 over 8000: 87 tiles of 125 k-steps, 42 us).  The input
// gradient is cut into `dsplit` fp32 slices of at least 8 k-steps where the
// modelled time with the slices' traffic is the least; core_split: the slices of
// the core's weight gradient.  Unsliced and so, both builds in turn on one card:
// the pair of 6 sequences of 300 tokens, width 192, 8000 words 40 -> 21 us (4
// slices) and the two-layer step, queued steps, 406 -> 380; 8 of 500, 256, 4096
// 33 -> 24 and 500 -> 495; 4 of 64, 128, 1024 8.7 -> 5.0 and 254 -> 250.
struct HeadPair {
  int tile = 0, split = 1, dsplit = 1;  // tile 0: the core's (its weight-gradient slices stay)
};
inline HeadPair wide_head_pair(int64_t N, int64_t V, int64_t d, int core_split) {
  const int64_t kd = (V + 63) / 64, kw = (N + 63) / 64;
  const double work = 4.0 * double(N) * double(V) * double(d) / 450e6 + 6.0;
  HeadPair best;
  double us = 1e30;
  for (int ds = 1; ds <= kWideMaxSplit && (ds == 1 || kd / ds >= 8); ds *= 2) {
    const int64_t kds = (kd + ds - 1) / ds;
    const double part = ds > 1 ? wide_part_us(N, d, ds) : 0.0;
    const double chain = 0.32 * double(std::max<int64_t>(kds, (kw + core_split - 1) / core_split)) + 4.0;
    if (const double t = std::max(work, chain) + part; t < us) {
      us = t;
      best = {0, core_split, ds};
    }
    const WideSplit m = mid_wgrad_split(V, d, N, us - part, 1, mid_tiles(N, d) * ds, kds);
    if (m.split) {
      us = m.us + part;
      best = {128, m.split, ds};
    }
  }
  // 256x256 tiles only where the input gradient alone fills the chip with them
  // (16384 x 512 over 32768: 768 us in 128 of them, 573 us in 512 of 128x128)
  if (wide_tiles(N, d) >= kWideCus) {
    const WideSplit w = wide_wgrad_split(V, d, N, us, 1, wide_tiles(N, d), kd);
    if (w.split) best = {256, w.split, 1};
  }
  return best;
}
// The core's split 64x64 weight gradient alone (512 x 2048 over 16384 rows:
// 75 us).
inline double wide_core_wgrad_us(int64_t M, int64_t N, int64_t K, int share) {
  return 2.0 * double(M) * double(N) * double(K) * share / 460e6 + 4.0;
}

}  // namespace erase
