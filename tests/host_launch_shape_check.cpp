// Host-side check of the launch shapes of 1x1 / FC rows: every length, from one row to very many, gets whole waves of a
// kernel that is built and that hold the row, with SQuant-C and without.
#include <cstdint>
#include <cstdio>
#include <initializer_list>

#include "squant_plan.h"

using namespace squant;

int main() {
  long bad = 0, shapes = 0;
  for (int64_t n = kMaxWaveCin + 1; n <= kMaxWideCin; ++n)
    for (int64_t rows : {1, 64, 300, 2000, 40000})
      for (int64_t half_bytes : {5, 6, 10, 12, 16}) {  // per weight, read and written
        const K1Shape s = k1_launch_shape((n + 3) / 4, rows, rows * n * half_bytes / 2, half_bytes >= 12);
        bad += !k1_built(s.nv, true) || s.threads % 64 != 0 || s.threads < 64 || s.threads > 1024 || (int64_t)s.nv * s.threads < (n + 3) / 4;
        ++shapes;
      }
  for (int64_t n = kMaxWaveCin + 1; n <= kMaxWideCin; ++n)
    for (bool aligned : {false, true}) {
      const int nv = k1_variant_nv(route_variant(1000, n, 1, aligned));
      bad += !k1_built(nv, false);
    }
  std::printf("shape_mismatches=%ld shapes=%ld\n", bad, shapes);
  return bad != 0;
}
