// Retained set of Eq. (9)-(10), one workgroup of 16 waves per sample.
//
// R starts as the pivots.  Stage i (pivot order) walks pivot i's ascending score
// list, skips tokens already in R and takes the first quota_i others: the threshold of
// Eq. (9) is set per pivot by the reduction ratio, i.e. by that quota.
//
// The scores are fp32 with absolute error <= tau, so a stage's outcome is certain
// only when the last score taken and the first one refused differ by more than
// 2*tau.  Decisions closer than that are settled in fp64 from the hidden-state
// rows, on (fp64 score, index).  The stages depend on each other, so the walk is
// a serial chain of LDS round trips; to keep it short the kernel speculates:
//   1. the stage lists are staged in LDS (in groups that fit);
//   2. one wave walks the stages in fp32 order, 128 or 256 list entries at a time (ranks by
//      ballots), committing what that order says, while the other waves move ahead of
//      it along the later stages' lists, past entries that are taken already (long quotas or
//      many stages: all waves together, kWideQuota);
//   3. the waves then look at the stages in parallel: a stage whose last key taken and
//      first key refused are
//      within 2*tau is uncertain, and its candidates within 2*tau of the boundary
//      are queued (who was a candidate is known from the per-token owner stage);
//   4. the waves re-score the queued (pivot, token) pairs in fp64, in parallel;
//   5. every uncertain stage is checked: if the fp64 order picks the same tokens
//      the speculation stands; at the first stage where it does not, that stage is
//      corrected, the later stages are undone and walked again.
// A boundary band that does not fit the queue or runs past the stored list (only
// with massive ties) is resolved by a block-wide sweep of the whole score row.
#pragma once
#include "common.hpp"

#include <type_traits>

namespace dart {

constexpr int kRetThreads = 1024;  // 16 waves for staging, the band phase and the fp64 re-scoring
constexpr int kRetWaves = kRetThreads / kWave;
// List entries staged in LDS at a time, as a 32-bit score image and a 16-bit token index each: the
// 32 lists of a 9216-token video sample (17424 entries) or the 16 lists of a 16384-token sample at
// one ninth (15.6 K) are staged in one go, and the walk reads the indices alone.
constexpr int kRetList = 18432;
static_assert(kRetList >= kMaxN, "a list has at most an entry per token: every stage is staged whole");
constexpr int kRetQ = 1024;      // band candidates awaiting an fp64 score
constexpr int kRetInFlight = 4;  // 16-byte pieces per row and lane in flight in the fp64 re-scoring
// Quotas from which the host takes the walk of all waves together (k_retain's WIDE): wave 0 alone
// takes about 0.25 us per stage and 0.1 us more for every 64 entries beyond 128, all waves 0.5 us
// whatever the length.  Order and retained set, wave 0 alone and all waves: 16 stages of quota 19 on
// 2880 tokens 16.6 and 19.3 us, 8 of quota 63 15.7 and 15.9, independent lists and equal ones alike; 8 of
// quota 70 15.7 and 16.0 (equal lists 16.3 and 16.1), of quota 100 15.9 and 16.4 (17.9 and 16.4).
// The helpers pass over some 64 taken entries per look, so with many stages and lists that are nearly
// the same wave 0 meets longer and longer heads: beyond kWideSlots slots in all the walk of all waves
// again (four samples of 9216 tokens, equal lists: 32 pivots of quota 32 30.3 and 33.6 us, 64 of 32 89
// and 78, 64 of 63 215 and 127; independent lists 25.6 and 33.0, 45.8 and 62, 73 and 81).
constexpr int kWideQuota = 64, kWideSlots = 2048;
constexpr unsigned char kOwnNone = 0xff, kOwnPivot = 0xfe;

struct RetainShared {
  // (what the walk touches comes first: within the 64 KiB that an LDS instruction's offset spans)
  // who took the token: a stage, kOwnPivot, or kOwnNone (the token is not retained); the last
  // kWave bytes stand for entries past a list's end (kOwnPivot: never a candidate)
  __attribute__((aligned(16))) unsigned char owner[kMaxN + kWave];
  int st_off[kMaxP];  // offset of the stage's list inside the sample's list region
  int st_len[kMaxP];
  // per stage: a list position at or before the last entry taken (where the walk began, every entry
  // before being taken by earlier stages; written by the walk alone); the position up to which the
  // helpers have found the list's entries taken (theirs alone, the walk reads it before its stage);
  // then the last key taken and the first refused
  int st_start[kMaxP];
  int st_ahead[kMaxP];
  unsigned long long st_kab[kMaxP][2];
  int st_qlo[kMaxP], st_qhi[kMaxP];
  unsigned char st_unc[kMaxP];
  int wcnt[kRetWaves];
  int qn, cnt, bad_first, fb_first;
  int walked;  // stages before this one are walked
  int piv[kMaxP];     // the pivots that are tokens
  double pl2[kMaxP];  // squared norms of the pivots, if given
  unsigned short lidx[kRetList];  // token indices of the staged entries (< kMaxN = 2^14)
  uint32_t lkey[kRetList];        // their score images
  double q_s64[kRetQ];
  int q_idx[kRetQ];
  unsigned char q_stage[kRetQ];
  unsigned char q_taken[kRetQ];
};

// A score that is not a number (a row or a pivot with an infinite or undefined element) counts as
// above every number.  With the pairs in a total order exactly `need` of a set have fewer than
// `need` before them, whatever the input holds: the retained set never outgrows its budget.
__device__ __forceinline__ double ordered_score(double s) { return s == s ? s : INFINITY; }

// (score, index) pairs compare lexicographically
__device__ __forceinline__ bool pair_less(double sa, int ja, double sb, int jb) {
  return sa < sb || (sa == sb && ja < jb);
}

// The retained set of sample b by one workgroup of kRetThreads threads.
// lists: per sample at P*row0, stage lists back to back (see k_order_scores).
// S: pivot-major scores.  X may be nullptr: then scores are taken as exact.
// pl2 [B*Ppad] (optional): fp64 squared norms of the pivots' rows, if this call computed them
// (the fp64 re-scoring then skips those products).
// keep: packed, ascending per sample.  cu_keep_out (optional) [B+1].
// scr_f64 [2*total_N] doubles: per-sample scratch at row0 (fallback sweep only).
// COH: S, lists and piv were written, and keep will be read, by other workgroups of this
// launch.  WIDE: how the stages are walked (see kWideQuota).
template <int DT, bool COH, bool WIDE>
__device__ __forceinline__ void retain_body(
    const Geo& g, int b, const float* S, const unsigned long long* lists, const int* piv,
    const void* X, int* keep, int* cu_keep_out, double* scr_f64, float two_tau,
    RetainShared& sh, const double* pl2 = nullptr) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const unsigned long long lt_mask = (1ull << lane) - 1ull;
  const Sample sm = sample_of(g, b);
  if (cu_keep_out && tid == 0) {
    cu_keep_out[b] = sm.keep0;
    if (b == g.B - 1) cu_keep_out[g.B] = sm.keep0 + sm.k;
  }
  if (sm.k == 0) return;
  const int n = sm.n, P = g.P, k = sm.k;
  const int esz = DT == kBF16 ? 2 : 4;
  const long rowbytes = g.ld * esz;
  const unsigned char* Xb =
      X ? static_cast<const unsigned char*>(X) + (long)sm.xrow * rowbytes : nullptr;
  const unsigned long long* glist = lists + (long)P * sm.row0;
  double* sweep_s64 = scr_f64 + sm.row0;                                   // fallback sweep
  int* sweep_idx = reinterpret_cast<int*>(scr_f64 + g.total_N + sm.row0);  // fallback sweep

  const Split sp(k, P, g.Pin);
  // stage constants in the lanes of every wave: lane i holds stage i's quota, list
  // length and list offset (the offsets are the prefix sums of the lengths)
  int quota_v = 0, len_v = 0;
  if (lane < P) {
    quota_v = sp.quota(lane);
    len_v = sp.stage_len(n, lane);
  }
  const int off_v = wave_excl_scan(len_v, lane);
  // Lists of the stages [first, group_hi) that fit in LDS together (the first one maybe
  // only in part); block-uniform arithmetic on the lane constants, no memory access.
  int group_hi = 0, group_base = 0, staged_total = 0;
  auto plan_group = [&](int first_any) {
    // (lane broadcasts by shuffle + readfirstlane: a readlane with a computed lane index did
    // not always compile here)
    const int first = __builtin_amdgcn_readfirstlane(first_any);  // block-uniform: keep it scalar
    group_base = __builtin_amdgcn_readfirstlane(__shfl(off_v, first, kWave));
    // a later stage joins the group while everything up to the end of its list fits; the list ends
    // grow with the stage, so the stages that fit are the lanes first .. group_hi-1
    const int rel_end = off_v + len_v - group_base;  // entries through stage `lane`
    const bool fits = lane >= first && lane < P && rel_end <= kRetList;
    group_hi = first + __builtin_amdgcn_readfirstlane(__popcll(__ballot(fits)));
    staged_total = __builtin_amdgcn_readfirstlane(__shfl(rel_end, group_hi - 1, kWave));
  };
  // a group moves in two halves of kStageLoads loads per thread (72 KiB in flight each)
  constexpr int kStageLoads = kRetList / kRetThreads / 2;
  unsigned long long staged[kStageLoads];
  auto load_half = [&](int h, int from) {
#pragma unroll
    for (int u = 0; u < kStageLoads; ++u) {
      const int t = (h * kStageLoads + u) * kRetThreads + from;
      staged[u] = t < staged_total ? ld_dev<COH>(&glist[group_base + t]) : 0ull;
    }
  };
  auto store_half = [&](int h, int from) {
#pragma unroll
    for (int u = 0; u < kStageLoads; ++u) {
      const int t = (h * kStageLoads + u) * kRetThreads + from;
      if (t < staged_total) {
        sh.lkey[t] = (uint32_t)(staged[u] >> 32);
        sh.lidx[t] = (unsigned short)staged[u];
      }
    }
  };

  // the first group's lists and the pivots are requested before LDS is cleared, so
  // the kernel waits for global memory once
  plan_group(0);
  load_half(0, tid);
  int my_pivot = -1;
  if (tid < g.Pin) my_pivot = ld_dev<COH>(&piv[b * P + tid]);  // pivots from outside hold no slot
  double my_pl2 = 0.0;
  if (pl2 && tid < P) my_pl2 = ld_dev<COH>(&pl2[b * g.Ppad + tid]);
  for (int t = tid; t < (n + 3) / 4; t += kRetThreads)
    reinterpret_cast<uint32_t*>(sh.owner)[t] = 0xffffffffu;
  if (tid < kWave) sh.owner[kMaxN + tid] = kOwnPivot;
  if (tid < g.Pin) sh.piv[tid] = my_pivot < 0 ? 0 : (my_pivot < n ? my_pivot : n - 1);
  if (pl2 && tid < P) sh.pl2[tid] = my_pl2;
  if (tid < P) {  // wave 0: its lanes hold the stage constants
    sh.st_len[tid] = len_v;
    sh.st_off[tid] = off_v;
  }
  store_half(0, tid);
  if (staged_total > kStageLoads * kRetThreads) {
    load_half(1, tid);
    store_half(1, tid);
  }
  __syncthreads();
  if (my_pivot >= 0 && my_pivot < n) sh.owner[my_pivot] = kOwnPivot;

  // row of stage st's pivot (the re-scoring waits for the rows alone: index and norm are in LDS)
  auto stage_pivot = [&](int st) -> const unsigned char* {
    if (st >= g.Pin)
      return static_cast<const unsigned char*>(g.E) + ((long)b * g.Pe + (st - g.Pin)) * g.lde * esz;
    return Xb + (long)sh.piv[st] * rowbytes;
  };
  // stages that take a token: with fewer slots than stages the last ones do not (a budget of the pivots
  // alone: none; walking them all the same made 65536 samples of at most 8 tokens 1467 us, 1396 before)
  const int stages = sp.q > 0 ? P : sp.r;
  int next = 0;  // first stage not yet final (block-uniform)
  while (next < stages) {
    if (next >= group_hi) {
      // (opaque, or the places of all loads are worked out ahead of the loop, where they cost every
      // call the registers of a second group: 21 spilled, 1 to 2 us)
      int from = tid;
      asm volatile("" : "+v"(from));
      plan_group(next);
      load_half(0, from);
      __syncthreads();  // nobody reads the old group any more
      store_half(0, from);
      if (staged_total > kStageLoads * kRetThreads) {
        load_half(1, from);
        store_half(1, from);
      }
    }
    if (tid == 0) {
      sh.qn = 0;
      sh.bad_first = group_hi;
      sh.fb_first = group_hi;
      sh.walked = next;
    }
    if (tid >= next && tid < group_hi) sh.st_start[tid] = sh.st_ahead[tid] = 0;
    __syncthreads();
    const int walk_end = group_hi < stages ? group_hi : stages;
    auto entry_of = [&](int i, int p) -> unsigned long long {  // entry p of stage i's list
      const int o = sh.st_off[i] - group_base + p;
      return ((unsigned long long)sh.lkey[o] << 32) | sh.lidx[o];
    };

    // ------------------------------------------------------------------ speculative walk
    // A stage depends on every earlier one, so the walk is as long as one wave's instruction
    // chain: wave 0 walks alone, kRun runs of 64 entries per stage straight-line and more only if
    // those do not fill the quota.  The LDS operations of a wave complete in order, so a stage's
    // marks are seen by the next stage's reads without a barrier; an entry costs one byte read (its
    // token's owner) and one byte written back; the next stage's indices are read ahead.  What
    // would make it long are the entries at the head of a list that earlier stages took
    // (near-duplicate pivots have nearly the same list, so stage i begins with most of what the i
    // stages before it took): the other waves keep moving st_ahead of the later stages past such
    // entries.  An entry once taken stays taken during the walk, so a position read late is only
    // less far ahead.  The walk reads a stage's position before it marks anything for that stage, so
    // what it reads passes over earlier stages' entries only.  A helper may store as late as it
    // likes: it may by then have passed over the stage's own entries, but nobody reads st_ahead of
    // a stage again, and st_start, which the boundary search below starts from, is not the helpers'.
    const auto lds_load = [](const int* p) {
      return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    const auto lds_store = [](int* p, int v) {
      __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    if constexpr (WIDE) {
      // Large quotas: all 16 waves in step, 1024 entries at a time, two barriers per stage.  The
      // next stage's entries travel together with the wave counts.
      auto first_tokens = [&](int st) -> int {
        const int o = __builtin_amdgcn_readlane(off_v, st) - group_base + tid;
        return sh.lidx[o < kRetList ? o : kRetList - 1];
      };
      int pre = first_tokens(next);
      for (int i = next; i < walk_end; ++i) {
        const int quota = __builtin_amdgcn_readlane(quota_v, i);
        const int len = __builtin_amdgcn_readlane(len_v, i);
        const int off = __builtin_amdgcn_readlane(off_v, i) - group_base;
        int taken = 0;
        for (int pos = 0; pos < len && taken < quota; pos += kRetThreads) {
          const int p = pos + tid;
          const bool busy = pos + (wave << 6) < len;  // wave-uniform: this wave has entries
          int j = kMaxN + lane;
          unsigned long long m = 0ull;
          if (busy) {
            if (p < len) j = pos == 0 ? pre : (int)sh.lidx[off + p];
            m = __builtin_amdgcn_ballot_w64(sh.owner[j] == kOwnNone);
          }
          if (lane == 0) sh.wcnt[wave] = __popcll(m);
          __syncthreads();
          if (pos == 0) pre = first_tokens(i + 1 < walk_end ? i + 1 : i);
          int x = lane < kRetWaves ? sh.wcnt[lane] : 0;  // inclusive prefix in lanes 0..15
          x += dpp_move<kDppShr1>(0, x);
          x += dpp_move<kDppShr2>(0, x);
          x += dpp_move<kDppShr4>(0, x);
          x += dpp_move<kDppShr8>(0, x);
          if (busy) {
            const int wv = __builtin_amdgcn_readfirstlane(wave);
            const int before = taken + (wv > 0 ? __builtin_amdgcn_readlane(x, wv > 0 ? wv - 1 : 0) : 0);
            const int r = before + __popcll(m & lt_mask);
            if (((m >> lane) & 1ull) != 0ull && r < quota) {
              sh.owner[j] = (unsigned char)i;
              if (r == quota - 1) sh.st_start[i] = p;  // the last one taken
            }
          }
          taken += __builtin_amdgcn_readlane(x, kRetWaves - 1);
          __syncthreads();  // the marks are visible before anyone tests them again
        }
        if (len == 0) pre = first_tokens(i + 1 < walk_end ? i + 1 : i);
      }
    } else if (wave == 0) {
      __builtin_amdgcn_s_setprio(3);
      int start_v = 0;  // lane i: where stage i's walk began
      auto walk = [&](auto runs) {
        constexpr int kRun = decltype(runs)::value;
        int tok[kRun];  // the stage's entries (token, or a byte past the tokens: no entry)
        int nxt[kRun];
        int pos = 0, ahead = 0;
        auto read_ahead = [&](int at, int off) {
#pragma unroll
          for (int c = 0; c < kRun; ++c) {
            const int o = off + at + c * kWave + lane;
            nxt[c] = sh.lidx[o < kRetList ? o : kRetList - 1];
          }
        };
        auto take_over = [&](int at, int len) {
#pragma unroll
          for (int c = 0; c < kRun; ++c)
            tok[c] = at + c * kWave + lane < len ? nxt[c] : kMaxN + lane;
        };
        int quota = __builtin_amdgcn_readlane(quota_v, next);
        int len = __builtin_amdgcn_readlane(len_v, next);
        int off = __builtin_amdgcn_readlane(off_v, next) - group_base;
        read_ahead(0, off);
        take_over(0, len);
        for (int i = next; i < walk_end; ++i) {
          int own[kRun];
#pragma unroll
          for (int c = 0; c < kRun; ++c) own[c] = sh.owner[tok[c]];
          const int in = i + 1 < walk_end ? i + 1 : i;
          const int quota_n = __builtin_amdgcn_readlane(quota_v, in);
          const int len_n = __builtin_amdgcn_readlane(len_v, in);
          const int off_n = __builtin_amdgcn_readlane(off_v, in) - group_base;
          const int pos_n = __builtin_amdgcn_readfirstlane(ahead);
          read_ahead(pos_n, off_n);
          ahead = lds_load(&sh.st_ahead[i + 2 < walk_end ? i + 2 : in]);
          start_v = lane == i ? pos : start_v;
          int taken = 0;  // candidates met so far
#pragma unroll
          for (int c = 0; c < kRun; ++c) {
            const unsigned long long m = __builtin_amdgcn_ballot_w64(own[c] == kOwnNone);
            const int r = __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                    __builtin_amdgcn_mbcnt_lo((unsigned)m, taken));
            sh.owner[tok[c]] = (unsigned char)(own[c] == kOwnNone && r < quota ? i : own[c]);
            taken += __popcll(m);
          }
          for (int p = pos + kRun * kWave; p < len && taken < quota; p += kWave) {
            const int j = p + lane < len ? (int)sh.lidx[off + p + lane] : kMaxN + lane;
            const bool cand = sh.owner[j] == kOwnNone;
            const unsigned long long m = __builtin_amdgcn_ballot_w64(cand);
            const int r = __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                    __builtin_amdgcn_mbcnt_lo((unsigned)m, taken));
            if (cand && r < quota) sh.owner[j] = (unsigned char)i;
            taken += __popcll(m);
          }
          lds_store(&sh.walked, i + 1);
          pos = pos_n;
          quota = quota_n;
          len = len_n;
          off = off_n;
          take_over(pos, len);
        }
      };
      // runs that usually fill the quota: about a third of the entries past st_ahead are taken
      if (sp.q < 40) walk(std::integral_constant<int, 2>{});
      else walk(std::integral_constant<int, 4>{});
      if (lane >= next && lane < walk_end) sh.st_start[lane] = start_v;
      __builtin_amdgcn_s_setprio(0);
    } else {
      // (A wave leaves when its last stage is the walk's next or is walked: the walk waits for
      // nobody.  It sleeps between looks: the LDS is the walk's.)
      const int last = next + wave - 1 + (walk_end - next - wave) / (kRetWaves - 1) * (kRetWaves - 1);
      bool moved = true;
      for (int seen = -1; next + wave - 1 < walk_end;) {
        const int walked = __builtin_amdgcn_readfirstlane(lds_load(&sh.walked));
        if (last <= walked + 1) break;
        if (walked == seen && !moved) {
          __builtin_amdgcn_s_sleep(4);
          continue;
        }
        seen = walked;
        moved = false;
        for (int i = next + wave - 1; i < walk_end; i += kRetWaves - 1) {
          const int len = __builtin_amdgcn_readlane(len_v, i);
          const int off = __builtin_amdgcn_readlane(off_v, i) - group_base;
          if (i <= walked + 1) continue;  // (the next two stages' positions have been read already)
          const int at = __builtin_amdgcn_readfirstlane(lds_load(&sh.st_ahead[i]));
          const int p = at + lane;
          const int j = p < len ? (int)sh.lidx[off + p] : 0;
          const unsigned char own = *(volatile unsigned char*)&sh.owner[j];
          const unsigned long long free_m = __ballot(p >= len || own == kOwnNone);
          const int step = free_m ? __builtin_ctzll(free_m) : kWave;
          if (step > 0) {
            if (lane == 0) lds_store(&sh.st_ahead[i], at + step);
            moved = true;
          }
        }
        __builtin_amdgcn_s_sleep(1);
      }
    }
    __syncthreads();

    // ------------------------------------------------------------------ uncertain stages
    // wave w looks at stages next+w, next+w+16, ...; owner is only read here
    for (int i = next + wave; i < walk_end; i += kRetWaves) {
      bool unc = false;
      uint32_t lo_m = 0, hi_m = 0;
      int pa = -1;  // list position of the last entry taken
      if (Xb && sp.quota(i) > 0) {
        // the last entry taken, and the first one refused: a candidate (not taken by an earlier
        // stage) that this stage did not take
        const int len = sh.st_len[i];
        int pb = -1;
        for (int p0 = sh.st_start[i]; p0 < len && pb < 0; p0 += kWave) {
          const int p = p0 + lane;
          const unsigned char own = p < len ? sh.owner[(uint32_t)entry_of(i, p)] : kOwnPivot;
          const unsigned long long mt = __ballot(own == (unsigned char)i);
          const unsigned long long mr = __ballot(own == kOwnNone || (own < kOwnPivot && (int)own > i));
          if (mt) pa = p0 + 63 - __builtin_clzll(mt);
          if (mr) pb = p0 + __builtin_ctzll(mr);
        }
        if (pa >= 0 && pb >= 0) {
          const unsigned long long ka = entry_of(i, pa), kb = entry_of(i, pb);
          const float fa = mono_inv((uint32_t)(ka >> 32)), fb = mono_inv((uint32_t)(kb >> 32));
          unc = !((fb - fa) > two_tau);
          lo_m = mono_of((fa - two_tau) + 0.0f);
          hi_m = mono_of((fb + two_tau) + 0.0f);
          if (lane == 0) {  // for the block-wide fallback
            sh.st_kab[i][0] = ka;
            sh.st_kab[i][1] = kb;
          }
        }
      }
      if (lane == 0) sh.st_unc[i] = unc ? 1 : 0;
      if (!unc) continue;
      const int len = sh.st_len[i];
      // reserves cnt queue slots, only if they fit (so every reserved slot gets written)
      auto reserve = [&](int cnt) -> int {
        int at = kRetQ + 1;
        if (lane == 0) {
          int old = sh.qn;
          while (old + cnt <= kRetQ) {
            const int seen = atomicCAS(&sh.qn, old, old + cnt);
            if (seen == old) {
              at = old;
              break;
            }
            old = seen;
          }
        }
        return __builtin_amdgcn_readfirstlane(at);
      };
      // Candidates of stage i = tokens no earlier stage owned.  Usually the band is a handful of
      // entries: one look at the 64 entries around the boundary that holds all of it, ends included.
      {
        const int w0 = pa - 31 > 0 ? pa - 31 : 0;
        const int p = w0 + lane;
        const unsigned long long e = p < len ? entry_of(i, p) : ~0ull;  // (past the end: above the band)
        const uint32_t key = (uint32_t)(e >> 32);
        const unsigned char own = p < len ? sh.owner[(uint32_t)e] : kOwnPivot;
        const unsigned long long below = __ballot(key < lo_m), above = __ballot(key > hi_m);
        const bool whole_below = w0 == 0 || (below & 1ull) != 0ull;
        const bool whole_above = w0 + kWave <= len ? above != 0ull : len == n || __ballot(p < len && key > hi_m) != 0ull;
        const bool band = key >= lo_m && key <= hi_m && (own == kOwnNone || (own < kOwnPivot && (int)own >= i));
        const unsigned long long mb = __ballot(band);
        if (whole_below && whole_above) {
          const int cnt = __popcll(mb);
          const int qlo = reserve(cnt);
          if (qlo + cnt > kRetQ) {
            if (lane == 0) atomicMin(&sh.fb_first, i);
            continue;
          }
          if (band) {
            const int slot = qlo + __popcll(mb & lt_mask);
            sh.q_idx[slot] = (int)(uint32_t)e;
            sh.q_stage[slot] = (unsigned char)i;
            sh.q_taken[slot] = own == (unsigned char)i ? 1 : 0;
          }
          if (lane == 0) {
            sh.st_qlo[i] = qlo;
            sh.st_qhi[i] = qlo + cnt;
          }
          continue;
        }
      }
      // first list position whose key reaches the band (64-ary search on the sorted keys)
      int lo_pos = 0, span = len;
      while (span > kWave) {
        const int stride = (span + kWave - 1) / kWave;
        const int p = lo_pos + lane * stride;
        const bool below = p < len && p < lo_pos + span &&
                           (uint32_t)(entry_of(i, p) >> 32) < lo_m;
        const int m = __popcll(__ballot(below));
        if (m > 0) lo_pos += (m - 1) * stride;
        span = stride;
      }
      auto scan = [&](int qbase) -> int {
        int cnt = 0;
        bool closed = false;
        for (int p0 = lo_pos; p0 < len && !closed; p0 += kWave) {
          const int p = p0 + lane;
          const unsigned long long e = p < len ? entry_of(i, p) : 0ull;
          const uint32_t key = (uint32_t)(e >> 32), idx = (uint32_t)e;
          const unsigned char own = p < len ? sh.owner[idx] : kOwnPivot;
          const bool band = p < len && key >= lo_m && key <= hi_m &&
                            (own == kOwnNone || (own < kOwnPivot && (int)own >= i));
          const unsigned long long mb = __ballot(band);
          if (qbase >= 0 && band) {
            const int slot = qbase + cnt + __popcll(mb & lt_mask);
            sh.q_idx[slot] = (int)idx;
            sh.q_stage[slot] = (unsigned char)i;
            sh.q_taken[slot] = own == (unsigned char)i ? 1 : 0;
          }
          cnt += __popcll(mb);
          closed = __ballot(p < len && key > hi_m) != 0ull;
        }
        return closed ? cnt : -1 - cnt;  // negative: the band reached the end of the list
      };
      int cnt = scan(-1);
      const bool open = cnt < 0 && len < n;  // the band may run past the stored list
      cnt = cnt < 0 ? -1 - cnt : cnt;
      const int qlo = open ? kRetQ + 1 : reserve(cnt);
      if (qlo + cnt > kRetQ) {
        // too many ties for the queue (or an open band): leave it to the block-wide sweep
        if (lane == 0) atomicMin(&sh.fb_first, i);
        continue;
      }
      scan(qlo);
      if (lane == 0) {
        sh.st_qlo[i] = qlo;
        sh.st_qhi[i] = qlo + cnt;
      }
    }
    __syncthreads();

    // ------------------------------------------------------------------ fp64 scores of the queue
    // block-uniform values read from LDS are made scalar explicitly: they end up as lane
    // indices of readlane, which must be scalar registers
    const int fb_first = __builtin_amdgcn_readfirstlane(sh.fb_first);
    const int qn = __builtin_amdgcn_readfirstlane(sh.qn);
    for (int q = wave; q < qn; q += kRetWaves) {  // a pair per wave: 16 row pairs in flight
      const int st = sh.q_stage[q];
      if (st >= fb_first) continue;  // will be walked again anyway
      const unsigned char* prow = stage_pivot(st);
      const unsigned char* xrow = Xb + (long)sh.q_idx[q] * rowbytes;
      const double s0 =
          pl2 ? row_cosine_f64<DT, true, kRetInFlight>(prow, xrow, g.D, lane, sh.pl2[st])
              : row_cosine_f64<DT, false, kRetInFlight>(prow, xrow, g.D, lane);
      if (lane == 0) sh.q_s64[q] = ordered_score(s0);
    }
    __syncthreads();

    // ------------------------------------------------------------------ check the speculation
    // the fp64 order agrees with the fp32 order iff the largest pair taken is below
    // the smallest pair refused
    for (int i = next + wave; i < walk_end && i < fb_first; i += kRetWaves) {
      if (!sh.st_unc[i]) continue;
      const int qlo = sh.st_qlo[i], qhi = sh.st_qhi[i];
      if (qhi - qlo <= 16) {  // few: a candidate per lane against each of the others
        const int q = qlo + lane;
        const bool mine = q < qhi && sh.q_taken[q] != 0;
        const double s = q < qhi ? sh.q_s64[q] : 0.0;
        const int j = q < qhi ? sh.q_idx[q] : 0;
        bool wrong = false;
        for (int o = qlo; o < qhi; ++o)
          wrong |= mine && sh.q_taken[o] == 0 && !pair_less(s, j, sh.q_s64[o], sh.q_idx[o]);
        if (__ballot(wrong) != 0ull && lane == 0) atomicMin(&sh.bad_first, i);
        continue;
      }
      double mt_s = -INFINITY, mu_s = INFINITY;
      int mt_j = -1, mu_j = 0x7fffffff;
      for (int q = qlo + lane; q < qhi; q += kWave) {
        const double s = sh.q_s64[q];
        const int j = sh.q_idx[q];
        if (sh.q_taken[q]) {
          if (pair_less(mt_s, mt_j, s, j)) { mt_s = s; mt_j = j; }
        } else {
          if (pair_less(s, j, mu_s, mu_j)) { mu_s = s; mu_j = j; }
        }
      }
#define DART_PAIR_STEP(J)                                                                      \
  {                                                                                            \
    const double s1 = lane_xor<J>(mt_s, lane), s2 = lane_xor<J>(mu_s, lane);                   \
    const int j1 = lane_xor<J>(mt_j, lane), j2 = lane_xor<J>(mu_j, lane);                      \
    if (pair_less(mt_s, mt_j, s1, j1)) { mt_s = s1; mt_j = j1; }                               \
    if (pair_less(s2, j2, mu_s, mu_j)) { mu_s = s2; mu_j = j2; }                               \
  }
      DART_PAIR_STEP(32) DART_PAIR_STEP(16) DART_PAIR_STEP(8) DART_PAIR_STEP(4) DART_PAIR_STEP(2)
      DART_PAIR_STEP(1)
#undef DART_PAIR_STEP
      if (!pair_less(mt_s, mt_j, mu_s, mu_j) && lane == 0) atomicMin(&sh.bad_first, i);
    }
    __syncthreads();
    const int bad = __builtin_amdgcn_readfirstlane(sh.bad_first);
    if (bad >= walk_end && fb_first >= walk_end) {
      next = walk_end;  // everything stands
      continue;
    }
    if (bad < fb_first) {
      // fp64 picks other tokens at stage `bad`: undo the later stages, correct this one
      for (int j = tid; j < n; j += kRetThreads) {
        const unsigned char o = sh.owner[j];
        if (o < kOwnPivot && (int)o > bad) sh.owner[j] = kOwnNone;
      }
      const int qlo = sh.st_qlo[bad], qhi = sh.st_qhi[bad];
      int need = 0;
      for (int q = qlo; q < qhi; ++q) need += sh.q_taken[q];
      __syncthreads();
      for (int q = qlo + tid; q < qhi; q += kRetThreads) {
        const double s = sh.q_s64[q];
        const int j = sh.q_idx[q];
        int beaten = 0;
        for (int o = qlo; o < qhi && beaten < need; ++o)
          beaten += pair_less(sh.q_s64[o], sh.q_idx[o], s, j) ? 1 : 0;
        const bool chosen = beaten < need;
        if (sh.q_taken[q] && !chosen) sh.owner[j] = kOwnNone;
        if (!sh.q_taken[q] && chosen) sh.owner[j] = (unsigned char)bad;
      }
      next = bad + 1;
      __syncthreads();
      continue;
    }

    // ------------------------------------------------------------------ block-wide fallback
    {
      // stage i and everything after it is taken back; stage i is decided on the
      // whole score row, then the walk goes on from i+1
      const int i = fb_first;
      for (int j = tid; j < n; j += kRetThreads) {
        const unsigned char o = sh.owner[j];
        if (o < kOwnPivot && (int)o >= i) sh.owner[j] = kOwnNone;
      }
      const int quota = sp.quota(i);
      const float lo = mono_inv((uint32_t)(sh.st_kab[i][0] >> 32)) - two_tau;
      const float hi = mono_inv((uint32_t)(sh.st_kab[i][1] >> 32)) + two_tau;
      const float* Srow = S + (long)P * sm.row0 + (long)i * n;
      if (tid == 0) sh.cnt = 0;
      __syncthreads();
      int n_in = 0;
      for (int j = tid; j < n; j += kRetThreads) {
        if (sh.owner[j] != kOwnNone) continue;
        const float s = ld_dev<COH>(&Srow[j]) + 0.0f;
        if (s < lo) {  // below the band: certainly among the quota lowest
          sh.owner[j] = (unsigned char)i;
          ++n_in;
        } else if (s <= hi) {
          sweep_idx[atomicAdd(&sh.cnt, 1)] = j;
        }
      }
      n_in = wave_sum(n_in);
      if (lane == 0) sh.wcnt[wave] = n_in;
      __syncthreads();
      int need = quota;
#pragma unroll
      for (int w = 0; w < kRetWaves; ++w) need -= sh.wcnt[w];
      const int nU = sh.cnt;
      const unsigned char* prow = stage_pivot(i);
      const double pp_i = pl2 ? sh.pl2[i] : 0.0;
      for (int u = wave; u < nU; u += kRetWaves) {
        const unsigned char* xrow = Xb + (long)sweep_idx[u] * rowbytes;
        const double s64 = pl2 ? row_cosine_f64<DT, true, kRetInFlight>(prow, xrow, g.D, lane, pp_i)
                               : row_cosine_f64<DT, false, kRetInFlight>(prow, xrow, g.D, lane);
        if (lane == 0) sweep_s64[u] = ordered_score(s64);
      }
      __syncthreads();
      for (int u = tid; u < nU; u += kRetThreads) {
        const double su = sweep_s64[u];
        const int ju = sweep_idx[u];
        int beaten = 0;
        for (int o = 0; o < nU && beaten < need; ++o)
          beaten += pair_less(sweep_s64[o], sweep_idx[o], su, ju) ? 1 : 0;
        if (beaten < need) sh.owner[ju] = (unsigned char)i;
      }
      next = i + 1;
      __syncthreads();
    }
  }
  __syncthreads();

  // emit the retained indices in ascending order: a thread owns 4, 8, 12 or 16 consecutive tokens
  const int per = (n + 4 * kRetThreads - 1) / (4 * kRetThreads);  // groups of four tokens (uniform)
  const int j0 = tid * per * 4;
  uint32_t kept = 0u;  // bit r: token j0 + r is retained
  for (int q = 0; q < per; ++q) {
    if (j0 + 4 * q < n) {  // (the bytes past the last token were cleared to kOwnNone with it)
      const uint32_t o4 = reinterpret_cast<const uint32_t*>(sh.owner)[tid * per + q];
#pragma unroll
      for (int r = 0; r < 4; ++r)
        kept |= ((o4 >> (8 * r)) & 0xffu) != kOwnNone ? 1u << (4 * q + r) : 0u;
    }
  }
  const int mine = __popc(kept);
  int off = wave_excl_scan(mine, lane);
  const int wtotal = __builtin_amdgcn_readlane(off + mine, 63);
  if (lane == 0) sh.wcnt[wave] = wtotal;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kRetWaves; ++w) off += w < wave ? sh.wcnt[w] : 0;
  int* out = keep + sm.keep0;
  for (; kept && off < k; ++off) {  // (never more than the budget: the next sample's rows follow)
    st_dev<COH>(out + off, j0 + __ffs(kept) - 1);
    kept &= kept - 1;
  }
}

// grid: B blocks of kRetThreads: block b builds the retained set of sample b.
template <int DT, bool WIDE>
__global__ __launch_bounds__(kRetThreads) void k_retain(
    Geo g, const float* __restrict__ S, const unsigned long long* __restrict__ lists,
    const int* __restrict__ piv, const void* __restrict__ X, int* __restrict__ keep,
    int* __restrict__ cu_keep_out, double* __restrict__ scr_f64, float two_tau,
    const double* __restrict__ pl2) {
  __shared__ RetainShared sh;
  retain_body<DT, false, WIDE>(g, blockIdx.x, S, lists, piv, X, keep, cu_keep_out, scr_f64,
                                 two_tau, sh, pl2);
}

}  // namespace dart
