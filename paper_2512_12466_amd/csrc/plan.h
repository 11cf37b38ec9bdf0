// Plans of the library's calls that follow from sizes and parameters alone.
// Plain C++ (no HIP), so that host programs can check them at sizes that no
// device run reaches.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

namespace nrt {

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
