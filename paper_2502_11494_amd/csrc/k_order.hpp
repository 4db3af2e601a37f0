// Score ordering: for every (sample, pivot) row of the score matrix, the lowest
// scores in ascending (score, index) order -- as many as stage i of the retained-set
// construction (Eq. 9-10) can possibly look at: the slots filled once stage i is
// done, plus one entry beyond to measure the margin of the stage's last decision.
#pragma once
#include "common.hpp"
#include "k_select.hpp"

namespace dart {

// What makes a value-linear histogram between the lowest and the highest score too coarse are the few scores
// far above the rest (tokens like the pivot), and those are never wanted.  The threads' lowest scores
// bound the want-th lowest from above: if they form at least `want` groups, the highest of the groups'
// minima is reached by `want` scores (of the second lowest of every thread: by twice as many as there
// are threads).  So the range ends there, every wanted score lies in it, and of its 1024 buckets one holds
// a few keys: the bucket that completes `want` ends the selection, prefix sums give every bucket's
// place, and a key finds its rank among the keys of its own bucket (five barriers; collect_sorted's
// way with its two histograms has twelve: lists of multi-crop 7.4 us, now 5.4, of sixteen 576-token images
// 5.8 and 4.9, of video 10.9 and 7.5, of 32 packed samples of up to 16384 tokens 25 and 18).
// Scores far below the rest (rows of zeros, say) crowd the others into a few buckets all the same.  If a
// selected bucket holds more than kOrderRefine keys, the selected ones are counted once more, in buckets of
// their own number: a coarse bucket is divided into as many parts as its share of the keys.  What still
// shares a bucket then has equal scores as a rule (copies of a row): up to kOrderTies such groups of any
// size are ranked by a bit per index.  Groups of more than kOrderCrowd different scores, more groups, and
// scores that are not numbers leave the list to collect_sorted.  (Ordering and retained set on given scores,
// 0.5 % of them zeros below a narrow rest, by collect_sorted, by cutting the range at the selected buckets
// first, and this way: eight samples of 2880 24.1, 28.2 and 17.0 us, four of 9216 60, 73 and 27.6, of 16384
// 107, 122 and 33; a tenth of the tokens equal 20.1, 23.8 and 17.4, 41, 50 and 27.9, 63, 76 and 33.5; two
// clusters, where the cut is enough, 18.9, 16.0 and 16.6, 27.1, 24.8 and 26.0, 33, 28.9 and 30.0.)
constexpr int kOrderRefine = 24, kOrderCrowd = 64, kOrderTies = 8;
template <int THREADS>
struct OrderShared {
  uint32_t lo[THREADS / kWave], hi[THREADS / kWave];
  int total[THREADS / kWave];
  int parts[kSelBuckets];  // of a coarse bucket: its first fine bucket and, << 16, how many it has
  int tie_from[kOrderTies], tie_to[kOrderTies];
  int last[2], count[2], crowded[2], mixed;  // (of the first and the second count)
};

// v[e] belongs to index tid + e*THREADS; put(position, key) receives the `want` lowest (value, index) keys.
// False (on every thread, nothing put): not done, see above.
template <int THREADS, int PER, typename Put>
__device__ __forceinline__ bool order_lowest(const float (&v)[PER], int n, int want, int tid,
                                             SelectShared<THREADS, PER>& sh, OrderShared<THREADS>& os,
                                             const Put& put) {
  constexpr int kWaves = THREADS / kWave, kOwn = kSelBuckets / THREADS;  // (1 or 2 buckets per thread)
  const int lane = tid & 63, w = tid >> 6;
  const int ne = __builtin_amdgcn_readfirstlane((n + THREADS - 1) / THREADS);
  const uint32_t none = mono_of(INFINITY);
  float low = INFINITY;
#pragma unroll
  for (int e = 0; e < PER; ++e)
    if (e < ne && tid + e * THREADS < n) low = fminf(low, v[e]);
  const uint32_t lowest = mono_of(low);
  uint32_t top = lowest;
  const int holders = n < THREADS ? n : THREADS;  // threads with a score: the first ones
  if (want <= holders) {
    // groups of 1, 2, 4, 8 or 16 neighbouring threads, as large as leaves `want` of them
    if (holders >= 2 * want) top = least(top, dpp_move<kDppXor1>(top, top));
    if (holders >= 4 * want) top = least(top, dpp_move<kDppXor2>(top, top));
    if (holders >= 8 * want) top = least(top, lane_xor<4>((int)top, lane));
    if (holders >= 16 * want) top = least(top, dpp_move<kDppRor8>(top, top));
  } else {
    const bool second = 2 * (n - THREADS < THREADS ? n - THREADS : THREADS) >= want;
    float next = second ? INFINITY : -INFINITY;
    low = INFINITY;
#pragma unroll
    for (int e = 0; e < PER; ++e)
      if (e < ne && tid + e * THREADS < n) {
        next = second ? fminf(next, fmaxf(low, v[e])) : fmaxf(next, v[e]);
        low = fminf(low, v[e]);
      }
    top = mono_of(next);
  }
  top = top == none ? 0u : top;  // no score (or no second one): not one of them
  const uint32_t wave_lo = wave_min_u32(lowest), wave_hi = wave_max_u32(top);
  if (lane == 0) {
    os.lo[w] = wave_lo;
    os.hi[w] = wave_hi;
  }
#pragma unroll
  for (int q = 0; q < kOwn; ++q) sh.hist[tid + q * THREADS] = 0;
  if (tid == 0) {
    os.count[0] = os.count[1] = -1;
    os.crowded[0] = os.crowded[1] = 0;
    os.mixed = 0;
  }
  __syncthreads();
  const float lo = mono_inv(row_min_u32(os.lo[lane % kWaves]));
  const float hi = mono_inv(row_max_u32(os.hi[lane % kWaves]));
  const float scale = hi > lo ? (float)kSelBuckets / (hi - lo) : 0.f;
  // (both monotone in x; a product that is no number, of an infinite range, counts as the highest)
  auto coarse = [&](float x) -> int { return (int)fminf((x - lo) * scale, (float)(kSelBuckets - 1)); };
  auto fine = [&](float x, int d) -> int {
    const int p = os.parts[d], first = p & 0xffff, more = (p >> 16) - 1;
    return more <= 0 ? first : first + (int)fminf(fmaf(x - lo, scale, -(float)d) * (float)(more + 1), (float)more);
  };
  int h[kOwn], before_own, c, end_bucket;
  // Counts the keys of every bucket (of(e): that of the thread's e-th score if it is selected, else
  // kSelBuckets); c: keys up to end_bucket, which completes `want` (-1: none does).  Returns how many of
  // these buckets hold more than `limit`.
  auto tally = [&](auto of, int limit, int second) -> int {
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int d = of(e);
      if (d < kSelBuckets) atomicAdd(&sh.hist[d], 1);
    }
    __syncthreads();
    int mine = 0;
#pragma unroll
    for (int q = 0; q < kOwn; ++q) {
      h[q] = sh.hist[tid * kOwn + q];
      mine += h[q];
    }
    int run = wave_excl_scan(mine, lane);
    if (lane == 63) os.total[w] = run + mine;
    __syncthreads();
    run += row_sum(lane % kWaves < w && (lane & 15) < kWaves ? os.total[lane % kWaves] : 0);
    before_own = run;
#pragma unroll
    for (int q = 0; q < kOwn; ++q) {
      const int before = run;
      sh.hist[tid * kOwn + q] = before;  // where the bucket's keys start
      run += h[q];
      if (before < want && h[q] > limit) {
        const int t = atomicAdd(&os.crowded[second], 1);
        if (second && t < kOrderTies) {
          os.tie_from[t] = before;
          os.tie_to[t] = run;
        }
      }
      if (before < want && run >= want) {
        os.last[second] = tid * kOwn + q;
        os.count[second] = run;
      }
    }
    __syncthreads();
    c = __builtin_amdgcn_readfirstlane(os.count[second]);
    end_bucket = __builtin_amdgcn_readfirstlane(os.last[second]);
    return __builtin_amdgcn_readfirstlane(os.crowded[second]);
  };
  auto scatter = [&](auto of) {
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int d = of(e);
      if (d <= end_bucket)
        sh.buf[atomicAdd(&sh.hist[d], 1)] =
            ((unsigned long long)mono_of(v[e]) << 32) | (unsigned)(tid + e * THREADS);
    }
    __syncthreads();
  };
  // a cell up to the last bucket's now holds the end of its bucket's keys = the start of the next
  auto rank = [&](auto bucket, int longest) {
    for (int t = tid; t < c; t += THREADS) {
      const unsigned long long key = sh.buf[t];
      const int d = bucket(mono_inv((uint32_t)(key >> 32)));
      int at = d > 0 ? sh.hist[d - 1] : 0;
      const int end = sh.hist[d];
      if (end - at > longest) continue;
      for (int u = at; u < end; ++u) at += sh.buf[u] < key ? 1 : 0;
      if (at < want) put(at, key);
    }
  };
  auto coarse_of = [&](int e) -> int {
    return e < ne && tid + e * THREADS < n && v[e] <= hi ? coarse(v[e]) : kSelBuckets;
  };
  const int crowded = tally(coarse_of, kOrderRefine, 0);
  if (c < 0) return false;  // (block-uniform, as all of these)
  if (crowded == 0) {
    scatter(coarse_of);
    rank(coarse, kOrderRefine);
    return true;
  }
  // of a coarse bucket whose keys are the before-th to the run-th of c: the fine buckets of that share
  const int last = end_bucket;
  const float share = (float)kSelBuckets / (float)c;
#pragma unroll
  for (int q = 0; q < kOwn; ++q) {
    const int first = (int)fminf((float)before_own * share, (float)(kSelBuckets - 1));
    before_own += h[q];
    const int next = (int)fminf((float)before_own * share, (float)(kSelBuckets - 1));
    os.parts[tid * kOwn + q] = first | ((next - first) << 16);
    sh.hist[tid * kOwn + q] = 0;  // (its own cells: nobody else has looked at them)
  }
  __syncthreads();
  auto divided = [&](float x) -> int {
    const int d = coarse(x);
    return d <= last ? fine(x, d) : kSelBuckets;
  };
  // (all of a thread's buckets before it counts the first: each takes an access to LDS)
  int slot[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int d = coarse_of(e);
    const int f = fine(v[e], d < kSelBuckets ? d : 0);
    slot[e] = d <= last ? f : kSelBuckets;
  }
  auto slot_of = [&](int e) -> int { return slot[e]; };
  const int ties = tally(slot_of, kOrderCrowd, 1);
  if (c < 0 || ties > kOrderTies) return false;
  scatter(slot_of);
  for (int s = 0; s < ties; ++s) {
    const int from = os.tie_from[s], to = os.tie_to[s];
    const uint32_t value = (uint32_t)(sh.buf[from] >> 32);
    for (int t = from + tid; t < to; t += THREADS)
      if ((uint32_t)(sh.buf[t] >> 32) != value) os.mixed = 1;
  }
  if (ties > 0) {
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(os.mixed) != 0) return false;
  }
  rank(divided, kOrderCrowd);
  // equal scores: a bit per index, and for every 32 of them how many come before
  constexpr int kWords = kMaxN / 32;
  static_assert(2 * kWords <= kSelBuckets, "bits and counts take the buckets' place");
  for (int s = 0; s < ties; ++s) {
    const int from = os.tie_from[s], to = os.tie_to[s];
    __syncthreads();
    for (int t = tid; t < kWords; t += THREADS) sh.hist[t] = 0;
    __syncthreads();
    for (int t = from + tid; t < to; t += THREADS) {
      const uint32_t j = (uint32_t)sh.buf[t];
      atomicOr(&sh.hist[j >> 5], (int)(1u << (j & 31)));
    }
    __syncthreads();
    if (w == 0) {
      constexpr int kOf = kWords / kWave;
      int mine = 0;
      for (int q = 0; q < kOf; ++q) mine += __popc(sh.hist[lane * kOf + q]);
      int run = wave_excl_scan(mine, lane);
      for (int q = 0; q < kOf; ++q) {
        sh.hist[kWords + lane * kOf + q] = run;
        run += __popc(sh.hist[lane * kOf + q]);
      }
    }
    __syncthreads();
    for (int t = from + tid; t < to; t += THREADS) {
      const unsigned long long key = sh.buf[t];
      const uint32_t j = (uint32_t)key;
      const int at = from + sh.hist[kWords + (j >> 5)] +
                     __popc((uint32_t)sh.hist[j >> 5] & ((1u << (j & 31)) - 1u));
      if (at < want) put(at, key);
    }
  }
  return true;
}

// A list that order_lowest leaves, by collect_sorted.  (A function of its own: inlined, its sorting
// networks cost the kernel 70 to 136 spilled registers at 16 scores per thread.)
template <int THREADS, bool COH, int PER>
__device__ __attribute__((noinline)) void order_crowded(const float* row, int n, int want,
                                                        unsigned long long* out,
                                                        SelectShared<THREADS, PER>& sh) {
  const int tid = threadIdx.x;
  n = __builtin_amdgcn_readfirstlane(n);
  want = __builtin_amdgcn_readfirstlane(want);
  float v[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int j = tid + e * THREADS;
    v[e] = ld_dev<COH>(&row[j < n ? j : n - 1]) + 0.0f;
  }
  int first = 0;  // keys of the first sorted run (all of them unless the sort was split)
  collect_sorted<THREADS, true, PER>(v, n, want, tid, sh, &first);
  for (int t = tid; t < want; t += THREADS)
    st_dev<COH>(&out[t], t < first ? sh.buf[t] : sh.buf[THREADS + (t - first)]);
}

// The list of stage i of sample b, by one workgroup of THREADS (1024) threads.
// S: pivot-major scores.  lists: 64-bit (score image << 32 | index) entries; the
// region of sample b starts at P*row0(b) and holds the stage lists back to back
// (see list_offset).
// COH: S was written, and lists will be read, by other workgroups of this launch.
template <int THREADS, bool COH, int PER = kSelPerThread>
__device__ __forceinline__ void order_scores_body(const Geo& g, int b, int i, const float* S,
                                                  unsigned long long* lists,
                                                  SelectShared<THREADS, PER>& sh,
                                                  OrderShared<THREADS>& os) {
  constexpr int kSelThreads = THREADS;
  const int tid = threadIdx.x;
  const Sample sm = sample_of(g, b);
  if (sm.k == 0) return;
  const int n = sm.n;
  const Split sp(sm.k, g.P, g.Pin);
  const int want = sp.stage_len(n, i);
  if (want == 0) return;  // the stage takes nothing
  const float* row = S + (long)g.P * sm.row0 + (long)i * n;
  // (all loads before the first use, from clamped places: see select_pivots_body)
  float v[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int j = tid + e * kSelThreads;
    v[e] = ld_dev<COH>(&row[j < n ? j : n - 1]);
  }
#pragma unroll
  for (int e = 0; e < PER; ++e) v[e] += 0.0f;  // -0 and +0 compare equal
  // offset of this stage's list = sum of the earlier stages' lengths: lane s of every wave
  // computes stage s's length, a wave scan adds them up (no loop over the stages)
  const int len_v = (tid & 63) < g.P ? sp.stage_len(n, tid & 63) : 0;
  const int off_v = wave_excl_scan(len_v, tid & 63);
  unsigned long long* out = lists + (long)g.P * sm.row0 + __builtin_amdgcn_readfirstlane(__shfl(off_v, i, kWave));
  if (order_lowest<THREADS, PER>(v, n, want, tid, sh, os, [&](int at, unsigned long long key) {
        st_dev<COH>(&out[at], key);
      }))
    return;
  order_crowded<THREADS, COH, PER>(row, n, want, out, sh);
}

// grid: B*P blocks of THREADS (1024); block (b, i), the samples from the longest to the
// shortest where g.by_size says so.  PER*THREADS >= the longest sample.
// (Samples of at most 4096 tokens: eight waves to a SIMD, so that two workgroups share a compute unit.  Without
// the bound the call of order_crowded takes 102 scalar registers, which leaves seven: lists of 32 samples
// of 2880 tokens, 16 pivots, 7.8 us and 6.2 with it, of 512 of 1500, 8 pivots, 45.6 and 31.8.  Longer ones
// have no room in LDS, or spill.)
template <int THREADS, int PER>
__global__ __launch_bounds__(THREADS)
__attribute__((amdgpu_waves_per_eu(PER <= 4 ? 8 : 4))) void k_order_scores(
    Geo g, const float* __restrict__ S, unsigned long long* __restrict__ lists) {
  __shared__ SelectShared<THREADS, PER> sh;
  __shared__ OrderShared<THREADS> os;
  const int slot = blockIdx.x / g.P;
  const int b = g.by_size ? g.by_size[slot] : slot;
  order_scores_body<THREADS, false, PER>(g, b, blockIdx.x % g.P, S, lists, sh, os);
}

}  // namespace dart
