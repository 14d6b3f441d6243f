// Exhaustive check of the two-operation quotient of 16-bit weights: every significand of a weight and of an absmax of
// binary16 (those of bfloat16 are among them) and every qmax, against IEEE division.  Exponents do not matter: both
// sides scale with powers of two as long as nothing under- or overflows.
//
// Build: g++ -O2 -mfma -ffp-contract=off
#include <cstdint>
#include <cstdio>

#include "squant_arith.h"

int main() {
  long checked = 0, bad = 0;
  for (int bits = 2; bits <= 8; ++bits) {
    const float qmax = (float)((1 << (bits - 1)) - 1);
    for (int a = 0; a < 1024; ++a) {
      const float s = (1.0f + (float)a / 1024.0f) / qmax, r = 1.0f / s, rl = squant::reciprocal_low(s, r);
      for (int m = 0; m < 1024; ++m) {
        const float w = 1.0f + (float)m / 1024.0f;
        bad += squant::half_quotient(w, r, rl) != w / s;
        ++checked;
      }
    }
  }
  std::printf("half_quotients=%ld mismatches=%ld\n", checked, bad);
  return bad != 0;
}
