// Host-side proof by enumeration for refine_reciprocal (squant_arith.h): for every significand
// of s and every binary32 estimate r0 within one unit in the last place of 1/s, one step gives
// the correctly rounded reciprocal - except from the lower of the two estimates of the reciprocal
// of 2 - 2^-23, for which the step ends on a tie; the hardware's estimate there is the upper one
// (0x3f000001; test_reciprocal_of_the_largest_significand pins it on the GPU).  Scaling s by a power of two scales r0 and every
// intermediate value exactly while nothing leaves the normal range, so one binade is enough.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>

#include "squant_arith.h"

static float next(float v, int steps) {
  int32_t b;
  std::memcpy(&b, &v, 4);
  b += steps;
  std::memcpy(&v, &b, 4);
  return v;
}

int main() {
  long mismatches = 0, known = 0, estimates = 0;
  for (uint32_t sig = 0; sig < (1u << 23); ++sig) {
    const uint32_t bits = 0x3F800000u | sig;  // s in [1, 2)
    float s;
    std::memcpy(&s, &bits, 4);
    const float want = 1.0f / s;
    for (int d = -2; d <= 2; ++d) {
      const float r0 = next(want, d);
      // |r0 - 1/s| <= ulp(1/s), decided exactly: |r0 s - 1| <= ulp s, every term a multiple of 2^-48
      const double ulp = want == 1.0f ? 0x1p-23 : 0x1p-24;
      if (std::fabs((double)r0 * (double)s - 1.0) > ulp * (double)s) continue;
      ++estimates;
      const float got = squant::refine_reciprocal(s, r0);
      if (std::memcmp(&got, &want, 4) != 0) {
        if (bits == 0x3FFFFFFFu && r0 == 0.5f) ++known; else ++mismatches;
      }
    }
  }
  std::printf("estimates=%ld known=%ld reciprocal_mismatches=%ld\n", estimates, known, mismatches);
  return mismatches != 0 || known != 1;
}
