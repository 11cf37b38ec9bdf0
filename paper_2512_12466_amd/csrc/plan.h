// Plans of the library's calls that follow from sizes and parameters alone.
// Plain C++ (no HIP), so that host programs can check them at sizes that no
// device run reaches.
#pragma once

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <exception>
#include <thread>
#include <vector>

#include "nyxrt.h"

namespace nrt {

// Line slots of a wavefront's deposit table (trace.hip), by the type of its sums.
constexpr int kLog2LinesFp32 = 8, kLog2LinesFp64 = 7;

// The slot of a line in a wavefront's deposit table is the top log2_lines bits
// of (line * M mod 2^24).  A bundle of rays fills the lines of a few cells
// around it, so M should send nearby lines (line +- 1 along x, n/8 along y,
// n^2/8 along z) to different slots, which depends on n: of 64 multipliers,
// the one with the least overlap of neighbours, weighted by a Gaussian of 4
// cells.  An emulation of bundles on nine grids of 64^3 to 1024^3, 128 slots
// folded at a quarter: a step of the wavefront probes past a first slot
// 0.3 times with it, 0.8 times with the golden-ratio multiplier.
inline uint32_t line_multiplier(int n, int log2_lines) {
  constexpr int kReach = 5;
  const uint32_t slot = 0x1000000u >> log2_lines;
  double weight[2 * kReach * kReach + 1];
  for (int r = 0; r <= 2 * kReach * kReach; ++r) weight[r] = std::exp(-r / 32.0);
  // of |x| = 0, 4, 8, 12 cells
  const double along[4] = {1.0, std::exp(-0.5), std::exp(-2.0), std::exp(-4.5)};
  double best = INFINITY;
  uint32_t mul = 0, x = 0x9E3779B9u;
  for (int q = 0; q < 64; ++q) {
    x = x * 1664525u + 1013904223u;
    const uint32_t m = (x >> 8) | 1u;
    double score = 0.0;  // only grows: a multiplier past the best so far is left
    for (int dz = 0; dz <= kReach && score < best; ++dz)
      for (int dy = dz ? -kReach : 0; dy <= kReach; ++dy) {
        const int64_t cells = int64_t(n) * dy + int64_t(n) * n * dz;
        // rows that do not start on a line share one with both neighbours
        const bool aligned = cells % 8 == 0;
        for (int dx = dz || dy ? -1 : 1; dx <= (aligned ? 1 : 2); ++dx) {
          const uint32_t p = (uint32_t(cells >> 3) + uint32_t(dx)) * m & 0xffffffu;
          const uint32_t gap = p >= 0x800000u ? 0x1000000u - p : p;
          const int cx = 8 * dx - (aligned ? 0 : 4);
          if (gap < slot)
            score += double(slot - gap) * weight[dy * dy + dz * dz] * along[std::abs(cx) / 4];
        }
      }
    if (score < best) {
      best = score;
      mul = m;
    }
  }
  return mul;
}

// The multipliers of an n^3 grid for tables of FP32 and of FP64 sums.  The search
// takes 12 us of a host core, a pass of the no-allocation call a few hundred, so
// each grid size is searched once a process and kept: both are 24 bits, one word
// a size, written whole (threads that race find the same), no heap and no
// thread-local storage, whose first use in a thread allocates.
struct LineMultipliers {
  uint32_t fp32, fp64;
};
inline LineMultipliers line_multipliers(int n) {
  static std::atomic<uint64_t> known[4097];  // by n; 0: not searched (multipliers are odd)
  std::atomic<uint64_t>& of_n = known[n];
  uint64_t v = of_n.load(std::memory_order_relaxed);
  if (!v) {
    v = uint64_t(line_multiplier(n, kLog2LinesFp32)) << 32 | line_multiplier(n, kLog2LinesFp64);
    of_n.store(v, std::memory_order_relaxed);
  }
  return {uint32_t(v >> 32), uint32_t(v)};
}

// Launch parameters that the autotuner times, in order: the library's default,
// the ones in use (`now`), and a grid around them.  The first two are there
// because the default differs by level (zeros), which no fixed choice can say.
// Refill 64: a wavefront refills only once drained (the best where the rays of
// a run live equally long).
inline std::vector<nrt_tuning> tuning_candidates(const nrt_tuning& now, int max_blocks_per_cu) {
  std::vector<nrt_tuning> cand{nrt_tuning{0, 0, 0, now.graph}};
  auto add = [&](const nrt_tuning& t) {
    for (const nrt_tuning& c : cand)
      if (std::memcmp(&c, &t, sizeof(t)) == 0) return;
    cand.push_back(t);
  };
  add(now);
  const int most = std::max(1, max_blocks_per_cu);
  for (int refill : {8, 16, 32, 64})
    for (int claim : {0, 64, 256})
      for (int bpc : {0, std::max(1, most - 1)})
        if (bpc != most) add(nrt_tuning{refill, claim, bpc, now.graph});
  return cand;
}

// The smallest path length at which a ray of a level splits (Eq.
// split_criterion): Omega(l) = 4 pi / (12 4^l) and Omega_c = 1 / s^2, so a ray
// splits iff s*s > 1 / (N_min Omega(l)).  The rounded square is monotone in s,
// so the test is a comparison with the smallest s that passes it, found by
// bisection over the ordered bit patterns of the doubles from 0 to infinity
// (N_min Omega may overflow, which leaves s*s > 0, or its reciprocal may).
// Infinity if none passes.
inline double split_length(double n_min_ray, int level) {
  if (!(n_min_ray > 0.0)) return INFINITY;
  const double omega = (4.0 * M_PI) / (12.0 * std::ldexp(1.0, 2 * level));
  const double r2 = 1.0 / (n_min_ray * omega);
  uint64_t lo = 0, hi = uint64_t(0x7ff) << 52;  // 0 does not pass; infinity is the answer else
  while (hi - lo > 1) {
    const uint64_t mid = lo + (hi - lo) / 2;
    double s;
    std::memcpy(&s, &mid, sizeof(s));
    (s * s > r2 ? hi : lo) = mid;
  }
  double s;
  std::memcpy(&s, &hi, sizeof(s));
  return s;
}

// fn(lo, hi) over [0, count) on up to 16 threads; on this one alone below
// `least` items a thread, and for a thread that cannot be started, whether the
// system has none left or there is no memory for it (either would leave running
// threads behind an exception, which ends the process).  fn must not throw.
template <typename Fn>
void over_threads(int64_t count, int64_t least, Fn fn) {
  const int64_t most = std::max(1u, std::min(16u, std::thread::hardware_concurrency()));
  const int64_t nt = std::max<int64_t>(1, std::min(most, count / least));
  std::thread th[16];
  for (int64_t t = 1; t < nt; ++t) {
    try {
      th[t] = std::thread(fn, count * t / nt, count * (t + 1) / nt);
    } catch (const std::exception&) {
      fn(count * t / nt, count * (t + 1) / nt);
    }
  }
  fn(int64_t(0), count / nt);
  for (auto& x : th)
    if (x.joinable()) x.join();
}

// Bins per axis of the merge's overlap search in an n^3 box: none narrower than
// `reach` cells, the largest distance at which two bubbles overlap; 1 means no
// binning (every pair is tested).  `need(bins)` is the scratch that a number of
// bins takes, of `scratch` bytes.  At most 1290 an axis: 1290^3 bins are fewer
// than 2^31, so a bin's index fits the kernels' 32-bit integers and stays off
// the mark of a source without a bin; wider bins only hold more candidates.
template <typename Need>
inline int64_t merge_bins(int64_t n, double reach, size_t scratch, Need need) {
  int64_t nb = std::min<int64_t>(int64_t(std::floor(double(n) / reach)), 1290);
  if (nb < 3) return 1;
  while (nb > 1 && need(nb * nb * nb) > scratch) --nb;
  return nb < 3 ? 1 : nb;
}

}  // namespace nrt
