// Prints, for each line "cout cin elements aligned" on standard input, how the planner routes such a tensor: its family,
// and for the kernels that hold whole channels of small kernels in registers (families 5 and 9) the kernels and threads
// of a launch of its own.  With an argument "rows" the lines are "longest rows bytes wide" (wide: 1 for
// binary32 output) and the answer is the launch shape of 1x1 / FC rows with SQuant-C: vectors and threads.
#include <cstdint>
#include <cstdio>
#include <cstring>

#include "squant_plan.h"

using namespace squant;

int main(int argc, char** argv) {
  long long a, b, c, d;
  if (argc > 1 && std::strcmp(argv[1], "rows") == 0) {
    while (std::scanf("%lld %lld %lld %lld", &a, &b, &c, &d) == 4) {
      const K1Shape s = k1_launch_shape((a + 3) / 4, b, c, d != 0);
      std::printf("%d %d\n", s.nv, s.threads);
    }
    return 0;
  }
  while (std::scanf("%lld %lld %lld %lld", &a, &b, &c, &d) == 4) {
    const int family = tensor_family(a, b, c, d != 0);
    int kpt = 0;
    if (family == 9 || family == 5) {
      const int v = variant_of_family(family, b, c, d != 0);
      kpt = family == 5 ? ks_variant_kpt(v) : v == kK9x4 ? 4 : v == kK9x2 ? 2 : 1;
    }
    std::printf("%d %d %lld\n", family, kpt, kpt ? (long long)round_up64((b + kpt - 1) / kpt) : 0);
  }
  return 0;
}
