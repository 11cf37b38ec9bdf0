// Host check (test infrastructure) of the plans in csrc/plan.h, one check a
// name on the command line.  Built and run by tests/test_plan.py.
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <thread>

#include "plan.h"

#define CHECK(x)                                              \
  do {                                                        \
    if (!(x)) {                                               \
      std::printf("line %d: %s is false\n", __LINE__, #x);    \
      return 1;                                               \
    }                                                         \
  } while (0)

// allocations still allowed; negative: any number
static std::atomic<int> g_allowed{-1};
__attribute__((noinline)) void* operator new(size_t bytes) {
  if (g_allowed >= 0 && g_allowed-- == 0) {
    g_allowed = 0;
    throw std::bad_alloc();
  }
  if (void* p = std::malloc(bytes)) return p;
  throw std::bad_alloc();
}
__attribute__((noinline)) void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { operator delete(p); }

// every item once, also when there is memory for the first threads only
static int over_threads() {
  for (int64_t count : {0, 1, 99, 100, 1000, 1001, 4096})
    for (int allowed : {-1, 0, 1, 2, 5}) {
      std::vector<std::atomic<int>> seen(4096);
      std::atomic<int>* s = seen.data();
      g_allowed = allowed;
      nrt::over_threads(count, 100, [s](int64_t lo, int64_t hi) {
        for (int64_t q = lo; q < hi; ++q) ++s[q];
      });
      g_allowed = -1;
      for (int64_t q = 0; q < 4096; ++q) CHECK(seen[size_t(q)] == (q < count ? 1 : 0));
    }
  return 0;
}

// a bin's index and the mark of a source without a bin share 32 bits, and the
// pair kernel's arithmetic is in int
static int merge_bins() {
  for (int64_t n : {1, 2, 3, 8, 64, 129, 1024, 1290, 1291, 1293, 1300, 1400, 1625, 1626, 4096})
    for (double reach : {1.0, 1.001, 1.5, 2.25, 17.0, 100.0, 1e9}) {
      const size_t cells = size_t(n) * n * n;
      const size_t scratch = std::max(cells * 16, size_t(1) << 22);
      auto need = [](int64_t bins) { return size_t(bins) * 12 + 65536; };
      const int64_t nb = nrt::merge_bins(n, reach, scratch, need);
      CHECK(nb >= 1 && nb != 2);
      CHECK(nb * nb * nb < (int64_t(1) << 31) - 1);
      CHECK(nb == 1 || double(n) / double(nb) >= reach);   // bins wide enough
      CHECK(nb == 1 || need(nb * nb * nb) <= scratch);
      // and no fewer than there can be
      CHECK(nb >= 1290 || nb == 1 || double(n) / double(nb + 1) < reach ||
            need((nb + 1) * (nb + 1) * (nb + 1)) > scratch);
      CHECK(nb != 1 || n < 3 * reach || need(27) > scratch);
      // a wider bin's neighbours: coordinate -> bin is monotone and in range
      CHECK((n - 1) * nb / n < nb);
    }
  return 0;
}

// the smallest s whose rounded square passes the split test, over the accepted
// N_min (finite, >= 0)
static int split_length() {
  const double n_mins[] = {0.0,    5e-324, 1e-310, 1e-308, 1e-300, 1e-20, 0.05, 1.0, 2.0,
                           3.0,    4.0,    5.5,    64.0,   1e20,   1e300, 1e308, 1.71e308,
                           1.717e308, 1.75e308, 1.7976931348623157e308};
  for (double n_min : n_mins)
    for (int level = 0; level <= 14; ++level) {
      const double s = nrt::split_length(n_min, level);
      const double omega = (4.0 * M_PI) / (12.0 * std::ldexp(1.0, 2 * level));
      const double r2 = n_min > 0.0 ? 1.0 / (n_min * omega) : INFINITY;
      CHECK(s > 0.0 && (s == INFINITY) == (r2 == INFINITY));
      CHECK(s * s > r2 || s == INFINITY);
      const double below = std::nextafter(s, 0.0);
      CHECK(!(below * below > r2));
    }
  return 0;
}

// the default and the set in use are among the autotuner's candidates, each
// candidate once and within what nrt_set_tuning takes
static int tuning_candidates() {
  const nrt_tuning sets[] = {{0, 0, 0, 0}, {16, 128, 0, 2}, {64, 64, 3, 1}, {5, 65536, 2, 0}};
  for (const nrt_tuning& now : sets)
    for (int most : {0, 1, 3, 4}) {
      const auto cand = nrt::tuning_candidates(now, most);
      int dflt = 0, in_use = 0;
      for (size_t i = 0; i < cand.size(); ++i) {
        const nrt_tuning& t = cand[i];
        dflt += t.refill_min == 0 && t.claim == 0 && t.blocks_per_cu == 0;
        in_use += std::memcmp(&t, &now, sizeof(t)) == 0;
        CHECK(t.refill_min >= 0 && t.refill_min <= 64 && t.claim >= 0 && t.claim <= 65536 &&
              t.claim % 64 == 0 && t.blocks_per_cu >= 0 && t.blocks_per_cu <= 64);
        CHECK(t.graph == now.graph);
        for (size_t j = 0; j < i; ++j) CHECK(std::memcmp(&t, &cand[j], sizeof(t)) != 0);
      }
      CHECK(dflt == 1 && in_use == 1);
      CHECK(cand.size() >= 12);
    }
  return 0;
}

// the kept multipliers are the search's for every grid size, whatever threads
// ask first; and sizes that alternate are not searched again (the time of 2000
// pairs of calls against that of 200 searches)
static int line_multipliers() {
  int wrong[4] = {0, 0, 0, 0};
  std::thread th[4];
  for (int t = 0; t < 4; ++t)
    th[t] = std::thread([t, &wrong] {
      for (int k = 0; k < 4096; ++k) {
        const int n = t % 2 ? 4096 - k : 1 + k;
        const nrt::LineMultipliers m = nrt::line_multipliers(n);
        wrong[t] += m.fp32 != nrt::line_multiplier(n, nrt::kLog2LinesFp32) ||
                    m.fp64 != nrt::line_multiplier(n, nrt::kLog2LinesFp64) || m.fp32 % 2 == 0 ||
                    m.fp64 % 2 == 0 || m.fp32 >> 24 || m.fp64 >> 24;
      }
    });
  for (auto& x : th) x.join();
  CHECK(wrong[0] + wrong[1] + wrong[2] + wrong[3] == 0);
  using Clock = std::chrono::steady_clock;
  const auto t0 = Clock::now();
  uint32_t sum = 0;
  for (int k = 0; k < 2000; ++k)
    sum += nrt::line_multipliers(24).fp32 + nrt::line_multipliers(40).fp64;
  const auto t1 = Clock::now();
  for (int k = 0; k < 200; ++k) sum += nrt::line_multiplier(24 + k % 7, 7);
  const auto t2 = Clock::now();
  CHECK(t1 - t0 < t2 - t1);
  std::printf("%u\n", sum);  // uses the loops' results
  return 0;
}

int main(int argc, char** argv) {
  for (int a = 1; a < argc; ++a) {
    int bad = 1;
    if (!std::strcmp(argv[a], "merge_bins")) bad = merge_bins();
    if (!std::strcmp(argv[a], "split_length")) bad = split_length();
    if (!std::strcmp(argv[a], "tuning_candidates")) bad = tuning_candidates();
    if (!std::strcmp(argv[a], "line_multipliers")) bad = line_multipliers();
    if (!std::strcmp(argv[a], "over_threads")) bad = over_threads();
    if (bad) {
      std::printf("%s failed\n", argv[a]);
      return 1;
    }
  }
  return 0;
}
