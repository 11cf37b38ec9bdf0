// Plans of the library's calls that follow from sizes and parameters alone.
// Plain C++ (no HIP), so that host programs can check them at sizes that no
// device run reaches.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <vector>

#include "nyxrt.h"

namespace nrt {

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
