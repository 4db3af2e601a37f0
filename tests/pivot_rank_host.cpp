// The candidate search of pivot selection on the CPU: the kernel's own integer functions over groups
// that are formed with plain loops.  v: the norms in the order that selection wants them (negated for
// the largest first).  cand[j] = 1 for every candidate; returns how many.
#include <math.h>
#include <string.h>

#include "../paper_2502_11494_amd/csrc/pivot_rank.hpp"

static uint32_t image(float f) {
  uint32_t u;
  memcpy(&u, &f, 4);
  return u ^ ((u >> 31) ? 0xffffffffu : 0x80000000u);
}
static float value(uint32_t m) {
  const uint32_t u = m ^ ((m >> 31) ? 0x80000000u : 0xffffffffu);
  float f;
  memcpy(&f, &u, 4);
  return f;
}

extern "C" int candidates(const float* v, int n, int want, float tau, unsigned char* cand,
                          int* looks) {
  uint32_t group[dart::kPivGroups];
  const uint32_t none = image(INFINITY);
  int seen = 0;
  for (int g = 0; g < dart::kPivGroups; ++g) {
    float low = INFINITY;
    for (int t = 0; t < 4; ++t)
      for (int e = 0; e < 16; ++e) {
        const int j = dart::pivot_token(4 * g + t, e);
        if (j >= n) continue;
        ++seen;
        low = fminf(low, v[j]);
      }
    group[g] = image(low);
  }
  if (seen != n) return -1;  // every token belongs to one group
  uint32_t lo = none, hi = 0;
  for (uint32_t m : group) {
    lo = m < lo ? m : lo;
    hi = m != none && m > hi ? m : hi;
  }
  *looks = 0;
  const uint32_t bound = dart::rank_bound(lo, hi, none, want, [&](uint32_t m) {
    int c = 0;
    for (uint32_t x : group) c += x <= m;
    ++*looks;
    return c;
  });
  const float thr = dart::candidate_limit(value(bound), tau);
  int count = 0;
  for (int j = 0; j < n; ++j) count += cand[j] = v[j] <= thr;
  return count;
}
