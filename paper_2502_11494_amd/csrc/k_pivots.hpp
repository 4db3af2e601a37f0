// Pivot selection (Definition 1; Table 1 caption: the P tokens of largest
// criterion norm), one workgroup per sample.
//
// The fp32 norms carry a relative error of at most `tau`.  Every token whose fp32 norm is
// within that error of the P-th best could belong to the exact top P, so all of them
// are ranked by (fp64 norm, index).  The norm pass leaves the fp64 norms beside the fp32 ones (tau
// is a rounding then); where the caller brought fp32 norms, the candidates' rows are summed here.
// The score kernel divides by the squared Euclidean norms of the pivots: they too come from the norm
// pass if it read the hidden states, else from the pivots' rows.
#pragma once
#include "common.hpp"
#include "pivot_rank.hpp"

namespace dart {

constexpr int kPivLdsCand = 512;  // candidates whose fp64 norms fit in LDS

// PER values per thread, PER*1024 >= the longest sample.
constexpr int kPivWaves = kPivThreads / kWave;

template <int PER>
struct PivotShared {
  __attribute__((aligned(16))) uint32_t group[kPivGroups];
  int cand[kPivThreads * PER];  // token indices
  double c64[kPivLdsCand];
  double l2[kPivLdsCand];
  int chosen[kMaxP];  // EXACT: the pivots (-1: none)
  int nU;
  float thr;
};

// rank_bound over 256 values by one wave, lane l holding four: a step is four compares and their
// ballots.
__device__ __forceinline__ uint32_t rank_bound_of_256(const u32x4& v, int want) {
  const uint32_t none = mono_of(INFINITY);  // groups without a token: not part of the range
  uint32_t lo = none, hi = 0u;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    lo = v[c] < lo ? v[c] : lo;
    hi = v[c] != none && v[c] > hi ? v[c] : hi;
  }
  const int lane = threadIdx.x & 63;
#define DART_MINMAX_STEP(J)                                                        \
  {                                                                                \
    const uint32_t a = (uint32_t)lane_xor<J>((int)lo, lane), b = (uint32_t)lane_xor<J>((int)hi, lane); \
    lo = lo < a ? lo : a;                                                          \
    hi = hi > b ? hi : b;                                                          \
  }
  DART_MINMAX_STEP(1) DART_MINMAX_STEP(2) DART_MINMAX_STEP(4) DART_MINMAX_STEP(8)
  DART_MINMAX_STEP(16) DART_MINMAX_STEP(32)
#undef DART_MINMAX_STEP
  const uint32_t l = __builtin_amdgcn_readfirstlane(lo), h = __builtin_amdgcn_readfirstlane(hi);
  return rank_bound(l, h, none, want, [&](uint32_t m) {
    return __popcll(__builtin_amdgcn_ballot_w64(v.x <= m)) +
           __popcll(__builtin_amdgcn_ballot_w64(v.y <= m)) +
           __popcll(__builtin_amdgcn_ballot_w64(v.z <= m)) +
           __popcll(__builtin_amdgcn_ballot_w64(v.w <= m));
  });
}

// Pivot selection of sample b by one workgroup of kPivThreads threads.
// l1 [total_N] fp32 criterion norms; piv [B*P] (the first Pin entries of a sample are
// written, and the marks of the pivots from outside); pl2 [B*Ppad] squared L2 norms of the pivots'
// rows (0 for the other slots), or nullptr: nobody wants them.
// EXACT: l1d [total_N], the fp64 norms of the same rows (l1 is their rounding); l2sq [total_N], the
// squared L2 norms of the hidden states' rows, or nullptr: those of the pivots are summed here.
// Otherwise l1d [2*total_N] is scratch.
// COH: l1 was written, and piv / pl2 will be read, by other workgroups of this launch.
template <int DT, bool COH, int PER, bool EXACT>
__device__ __forceinline__ void select_pivots_body(
    const Geo& g, int b, const void* X, const void* C, int Dc, long ldc, const float* l1,
    int* piv, double* pl2, double* l1d, const double* l2sq, float tau, PivotShared<PER>& sh) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const Sample sm = sample_of(g, b);
  if (tid < g.Ppad) {
    if (pl2 && (tid < g.Pin || tid >= g.P || sm.k == 0)) st_dev<COH>(&pl2[b * g.Ppad + tid], 0.0);
    if (tid >= g.Pin && tid < g.P) st_dev<COH>(&piv[b * g.P + tid], -1 - (tid - g.Pin));
  }
  if (sm.k == 0) return;
  if (COH) stores_done();
  const int n = sm.n, P = g.Pin;  // pivots chosen among the tokens; stride of piv is g.P
  const float sign = g.mode == kMaxL1 ? -1.f : 1.f;  // "lowest" of -norm = largest norm

  // Candidates: every token that may belong to the exact top P.  The tokens form 256 groups of four
  // threads each (pivot_token); the P-th lowest of the groups' lowest values is reached by P tokens,
  // so with vsel at least that, {v <= vsel + 2.5 tau |vsel|} holds every token within the norm
  // pass's error of the P-th best: usually P and a handful more.  They are ranked in fp64 below, so
  // neither their order nor the exact P-th value is needed here.  (Two barriers; the histogram over
  // the block's value range that this replaces had six.)
  // (all loads before the first use, from clamped places: a load whose value is used under its
  // condition is waited for before the next one is issued, 0.3 us each)
  float v[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int j = pivot_token(tid, e);
    v[e] = ld_dev<COH>(&l1[sm.row0 + (j < n ? j : n - 1)]);
  }
  float low = INFINITY;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    v[e] = pivot_token(tid, e) < n ? sign * v[e] + 0.0f : INFINITY;
    low = fminf(low, v[e]);
  }
  low = fminf(low, lane_xor<1>(low, lane));
  low = fminf(low, lane_xor<2>(low, lane));
  if ((tid & 3) == 0) sh.group[tid >> 2] = mono_of(low);
  if (tid == 0) sh.nU = 0;
  if (EXACT && tid < P) sh.chosen[tid] = -1;
  const int esz = DT == kBF16 ? 2 : 4;
  __syncthreads();  // (and the zeros above are ordered before the pivots' norms below)
  if (w == 0) {  // (alone it takes half as long as with all waves beside it)
    const u32x4 g4 = reinterpret_cast<const u32x4*>(sh.group)[lane];
    const float vsel = mono_inv(rank_bound_of_256(g4, P));
    if (lane == 0) sh.thr = candidate_limit(vsel, tau);
  } else if (pl2) {
    // meanwhile the others sum the pivots from outside (a launch of their own takes 4.5 us)
    for (int e = w - 1; e < g.Pe; e += kPivWaves - 1) {
      double unused, q;
      row_l1_l2_f64<DT>(static_cast<const unsigned char*>(g.E) + ((long)b * g.Pe + e) * g.lde * esz,
                        g.D, lane, unused, q);
      if (lane == 0) st_dev<COH>(&pl2[b * g.Ppad + g.Pin + e], q);
    }
  }
  __syncthreads();
  const float thr = sh.thr;
  uint32_t hit = 0u;  // (few threads have one)
#pragma unroll
  for (int e = 0; e < PER; ++e) hit |= v[e] <= thr ? 1u << e : 0u;
  const double flip = g.mode == kMaxL1 ? -1.0 : 1.0;
  while (__builtin_amdgcn_ballot_w64(hit != 0u) != 0ull) {
    if (hit != 0u) {
      const int j = pivot_token(tid, __ffs(hit) - 1);
      hit &= hit - 1u;
      if (j < n) {
        const int u = atomicAdd(&sh.nU, 1);
        sh.cand[u] = j;
        if (EXACT && u < kPivLdsCand) {
          sh.c64[u] = flip * l1d[sm.row0 + j];
          if (l2sq) sh.l2[u] = l2sq[sm.row0 + j];
        }
      }
    }
  }
  __syncthreads();
  const int nU = sh.nU;  // 0 only if the norms are not numbers: then no pivot is written

  const unsigned char* Xb = static_cast<const unsigned char*>(X) + (long)sm.xrow * g.ld * esz;
  const bool in_lds = nU <= kPivLdsCand;
  double* c64 = in_lds ? sh.c64 : l1d + sm.row0;
  double* l2s = in_lds ? sh.l2 : l1d + g.total_N + sm.row0;
  if constexpr (!EXACT) {
    const unsigned char* Cb = static_cast<const unsigned char*>(C) + (long)sm.xrow * ldc * esz;
    for (int u = w; u < nU; u += kPivWaves) {  // a candidate per wave
      const int j = sh.cand[u];
      double a, q;
      row_l1_l2_f64<DT>(Cb + (long)j * ldc * esz, Dc, lane, a, q);
      if (C != X || Dc != g.D || ldc != g.ld) {
        double unused;
        row_l1_l2_f64<DT>(Xb + (long)j * g.ld * esz, g.D, lane, unused, q);
      }
      if (lane == 0) {
        c64[u] = g.mode == kMaxL1 ? -a : a;
        l2s[u] = q;
      }
    }
    __syncthreads();
  }
  // norm of candidate u (more candidates than the LDS holds: from the norm pass's array by token)
  auto norm_of = [&](int u, int j) { return !EXACT || in_lds ? c64[u] : flip * l1d[sm.row0 + j]; };
  auto choose = [&](int rank, int u, int j) {
    st_dev<COH>(&piv[b * g.P + rank], j);
    if (!pl2) return;
    if (!EXACT) {
      st_dev<COH>(&pl2[b * g.Ppad + rank], l2s[u]);
    } else if (l2sq) {
      st_dev<COH>(&pl2[b * g.Ppad + rank], in_lds ? sh.l2[u] : l2sq[sm.row0 + j]);
    } else {
      sh.chosen[rank] = j;
    }
  };
  // rank by (fp64 value, index); only ranks < P matter
  if (nU <= 2 * kWave) {
    // a wave per candidate: lane o compares candidates o and o + 64 with it, the ballots count
    const int o2 = lane + kWave;
    const bool on = lane < nU, on2 = o2 < nU;
    const double co = on ? c64[lane] : 0.0, co2 = on2 ? c64[o2] : 0.0;
    const int jo = on ? sh.cand[lane] : 0, jo2 = on2 ? sh.cand[o2] : 0;
    for (int u = w; u < nU; u += kPivWaves) {
      const double cu = c64[u];
      const int ju = sh.cand[u];
      int cnt = __popcll(__ballot(on && (co < cu || (co == cu && jo < ju))));
      if (nU > kWave) cnt += __popcll(__ballot(on2 && (co2 < cu || (co2 == cu && jo2 < ju))));
      if (lane == 0 && cnt < P) choose(cnt, u, ju);
    }
  } else {
    for (int u = tid; u < nU; u += kPivThreads) {
      const int ju = sh.cand[u];
      const double cu = norm_of(u, ju);
      int cnt = 0;
      for (int o = 0; o < nU && cnt < P; ++o) {
        const int jo = sh.cand[o];
        const double co = norm_of(o, jo);
        cnt += (co < cu || (co == cu && jo < ju)) ? 1 : 0;
      }
      if (cnt < P) choose(cnt, u, ju);
    }
  }
  if (EXACT && pl2 && l2sq == nullptr) {
    __syncthreads();
    for (int i = w; i < P; i += kPivWaves) {
      const int j = sh.chosen[i];
      if (j < 0) continue;
      double unused, q;
      row_l1_l2_f64<DT>(Xb + (long)j * g.ld * esz, g.D, lane, unused, q);
      if (lane == 0) st_dev<COH>(&pl2[b * g.Ppad + i], q);
    }
  }
}

// grid: B blocks of kPivThreads: block b selects the pivots of sample b.
// TWO: 64 registers, so that two workgroups share a compute unit (selection of 512 samples of 1500 tokens 8.0 us
// with the 68 registers the compiler takes by itself and 5.8 this way, of 300 of 2000 7.2 and 4.9).  Eight of
// them are spilled where rows are summed, so only for more samples than there are units: eight samples of
// 2880 with a separate criterion 5.0 us without and 5.6 with it.
template <int DT, int PER, bool EXACT, bool TWO>
__global__ __launch_bounds__(kPivThreads)
__attribute__((amdgpu_waves_per_eu(TWO ? 8 : 4))) void k_select_pivots(
    Geo g, const void* __restrict__ X, const void* __restrict__ C, int Dc, long ldc,
    const float* __restrict__ l1, int* __restrict__ piv, double* __restrict__ pl2,
    double* __restrict__ l1d, const double* __restrict__ l2sq, float tau) {
  __shared__ PivotShared<PER> sh;
  select_pivots_body<DT, false, PER, EXACT>(g, blockIdx.x, X, C, Dc, ldc, l1, piv, pl2, l1d, l2sq,
                                            tau, sh);
}

}  // namespace dart
