// Host-side check of next_key_below (squant_arith.h) in the selection it serves: TEAM lanes with NE
// keys each offer their largest key not yet taken, the largest offer of the team is taken and its lane
// moves on, until `need` keys are taken or none is left; a lane then flips its keys at or above the
// smallest one taken.  Compared with sorting, for keys of which none, some or all are 0, and for every
// `need` from 1 to more than there are keys.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <random>
#include <vector>

#include "squant_arith.h"

using namespace squant;

template <int TEAM, int NE>
long check(std::mt19937& rng, int rounds) {
  long bad = 0;
  for (int r = 0; r < rounds; ++r) {
    uint32_t key[TEAM][NE];
    std::vector<uint32_t> all;
    const int eligible = r % 4;  // 0: every key, 1: most, 2: half, 3: few
    const uint32_t spread = r % 3 == 0 ? 1u : r % 3 == 1 ? 64u : 1u << 22;  // equal, few levels, any
    for (int l = 0; l < TEAM; ++l)
      for (int e = 0; e < NE; ++e) {
        const uint32_t u = (1u << 22) - rng() % spread, index = (uint32_t)(4 * (l + (e >> 2) * TEAM) + (e & 3));
        const uint32_t dice = rng() % 8;
        const bool in = eligible == 0 || (eligible == 1 && dice != 0) || (eligible == 2 && dice < 4) || (eligible == 3 && dice == 0);
        key[l][e] = in ? (u << 8) | (255u - index) : 0u;
        if (in) all.push_back(key[l][e]);
      }
    std::sort(all.rbegin(), all.rend());
    for (uint32_t need = 1; need <= TEAM * NE + 1; ++need) {
      uint32_t offer[TEAM], taken[TEAM], left = need;
      for (int l = 0; l < TEAM; ++l) {
        offer[l] = *std::max_element(key[l], key[l] + NE);
        taken[l] = ~0u;
      }
      while (left > 0) {
        const uint32_t m = *std::max_element(offer, offer + TEAM);
        const bool take = m != 0;
        for (int l = 0; l < TEAM; ++l) {
          const uint32_t next = next_key_below(key[l], offer[l]);
          const bool mine = take && offer[l] == m;
          taken[l] = mine ? m : taken[l];
          offer[l] = mine ? next : offer[l];
        }
        left = take ? left - 1 : 0u;
      }
      const size_t want = std::min<size_t>(need, all.size());
      for (int l = 0; l < TEAM; ++l)
        for (int e = 0; e < NE; ++e) {
          const bool flips = key[l][e] >= taken[l];
          const bool should = key[l][e] != 0 && want > 0 && key[l][e] >= all[want - 1];
          bad += flips != should;
        }
    }
  }
  return bad;
}

int main() {
  std::mt19937 rng(7);
  long bad = check<4, 4>(rng, 600) + check<8, 4>(rng, 400) + check<16, 4>(rng, 200) + check<16, 8>(rng, 100) +
             check<16, 16>(rng, 60);
  std::printf("key_step_mismatches=%ld\n", bad);
  return bad != 0;
}
