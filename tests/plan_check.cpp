// Host check (test infrastructure) of the plans in csrc/plan.h, one check a
// name on the command line.  Built and run by tests/test_plan.py.
#include <cstdio>
#include <cstring>

#include "plan.h"

#define CHECK(x)                                              \
  do {                                                        \
    if (!(x)) {                                               \
      std::printf("line %d: %s is false\n", __LINE__, #x);    \
      return 1;                                               \
    }                                                         \
  } while (0)

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

int main(int argc, char** argv) {
  for (int a = 1; a < argc; ++a) {
    int bad = 1;
    if (!std::strcmp(argv[a], "merge_bins")) bad = merge_bins();
    if (bad) {
      std::printf("%s failed\n", argv[a]);
      return 1;
    }
  }
  return 0;
}
