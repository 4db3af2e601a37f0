// How pivot selection finds a bound of the P-th best norm: the plain integer part of it, which
// compiles for the host too, so that the number of candidates it leaves can be checked without a GPU.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define DART_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define DART_HOST_DEVICE inline
#endif

namespace dart {

// 1024 threads; four of them share a group of tokens.
constexpr int kPivThreads = 1024, kPivGroups = kPivThreads / 4;

// Token that thread tid holds in slot e; a sample of at most 256 tokens has one per group.  Groups
// should not mirror the order of the tokens: a group of every 256th token (this without the shift)
// holds the same place of every frame if a video's frames have 256 tokens, or a divisor of 256, and
// with norms that follow the place 32 groups reach no further than 32 places, each with all its
// frames: 1050 candidates for 32 pivots among 9216 tokens, 460 us for four such samples instead of
// 155.  So every run of 256 tokens is dealt with a shift of its own; it is quadratic because with a
// linear one another period takes the place of 256 (37 per run: 219).  At most 50 candidates for 32
// pivots over all periods up to 1500.
DART_HOST_DEVICE int pivot_token(int tid, int e) {
  const int run = 4 * e + (tid & 3);
  return run * kPivGroups + (((tid >> 2) - run * (11 * run + 37)) & (kPivGroups - 1));
}

// A bound of the want-th lowest of a set of values (order-preserving images of floats), at least
// that value: bisection between the lowest value and the highest, lo and hi, where count(m) says how
// many values are at most m.  It ends when at most one value too many is below the bound (six to ten
// steps as a rule) or at a range of kRankClose images, about the margin that the caller adds to
// the bound anyway, however far apart lo and hi are: an image is a floating-point number, and one zero
// among norms of thousands makes it 18 steps.  none if hi itself does not reach want values.
constexpr uint32_t kRankClose = 32;
template <typename Count>
DART_HOST_DEVICE uint32_t rank_bound(uint32_t lo, uint32_t hi, uint32_t none, int want,
                                     const Count& count) {
  uint32_t l = lo, h = hi;
  while (l < h && h - l >= kRankClose) {  // the bound is in [l, h]
    const uint32_t mid = l + ((h - l) >> 1);
    const int c = count(mid);
    if (c >= want) h = mid; else l = mid + 1;
    if (c == want || c == want + 1) break;  // close enough (h = mid)
  }
  return h == hi && count(h) < want ? none : h;
}

// Values up to this belong to the candidates: the bound and the norm pass's error tau on either
// side of it.  Everything if the bound is not a finite number (norms beyond the range of fp32, or
// fewer groups than pivots hold a number): the fp64 ranking decides.
DART_HOST_DEVICE float candidate_limit(float bound, float tau) {
  const float mag = bound < 0.f ? -bound : bound;
  return mag < __builtin_inff() ? bound + 2.5f * tau * mag : __builtin_inff();
}

}  // namespace dart
