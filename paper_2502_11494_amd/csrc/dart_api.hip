// Host side of the DART C ABI (include/dart.h): argument checks, workspace
// carving and kernel launches.  No allocation, no synchronisation except in
// dart_device_status.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <mutex>

#include "../../include/dart.h"
#include "common.hpp"
#include "k_fused.hpp"
#include "k_misc.hpp"
#include "k_norms.hpp"
#include "k_order.hpp"
#include "k_pivots.hpp"
#include "k_retain.hpp"
#include "k_scores.hpp"
#include "k_single.hpp"

using namespace dart;

// Scratch of dart_reduce_static: one copy per GPU, at an address of its own on each.  In host
// code this name is only a handle for hipGetSymbolAddress, never a device address.
constexpr size_t kStaticScratchBytes = size_t(32) << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

constexpr size_t kAlign = 256;
// Row strides (elements) are bounded so that rows * stride * element size stays far inside 64
// bits on the host and in the kernels' byte offsets.
constexpr int64_t kMaxLd = int64_t(1) << 24;
constexpr int kMaxB = 1 << 20;  // samples per call (grids and offset tables are sized by B)
inline size_t up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

struct Plan {
  Geo g;
  int esz;
  long keep_rows_bound;  // upper bound of the total number of retained rows
  int tiles_bound;       // upper bound of the number of score tiles (g.tile_rows rows each)
  // workspace offsets
  size_t o_status, o_cu_keep, o_tile_start, o_l1, o_piv, o_pl2, o_S, o_lists, o_scr_f64,
      o_l2, o_sync, o_nstart, o_sstart, o_gstart, o_by_size, total;
  bool fusable;  // the shape and modes the one-launch path covers (see reduce_impl)
  bool norms_given;  // this call's norm pass also leaves the squared token norms
  int ks_waves, ks_split;  // bf16 score kernel: waves per workgroup and groups of them (fp32: 0)
  int f32_groups;  // fp32 score tiles of 4 rows: groups of four pivots per workgroup
  unsigned long long seed; // DART_PIVOT_RANDOM: the seed of the draw
};

// Compute units of the current GPU looked up once per GPU.
int compute_units() {
  static std::mutex m;
  static int cached[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  std::lock_guard<std::mutex> lock(m);
  if (cached[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
    cached[dev] = n;
  }
  return cached[dev];
}

// ---- tile shape of the bf16 score kernel ----------------------------------------------------
// k_scores_ksplit takes any number of waves W per workgroup and splits the D-chunks over KS
// groups of them, so a tile has R = 16*W/KS rows.  Measured on the benchmark shapes the kernel
// runs at the speed of the busiest compute unit: about 6 TB/s for the chip as a whole (pivot
// chunks, served by L2, count about a fifth of their bytes), plus 48 GB/s for whatever rows
// the busiest unit holds beyond the average (the units take ceil(tiles/256) or one fewer tiles
// each), and never faster than a wave's chain of chunks (0.55 us each).  Tile heights that
// divide the batch evenly over the 256 units therefore win: 9 waves (144 rows) for four
// samples of 9216 tokens (47 us against 55 with 64-row tiles), 12 waves in 4 groups (48 rows)
// for sixteen of 576 (18 us against 27 for four workgroups per tile and a finishing pass).
// The candidates are the shapes instantiated below; (8, 8), 16-row tiles with a chain of an eighth of
// the chunks, is for batches of so few rows that nothing but the chain counts (whole step against
// the 32-row tiles of (8, 4): one frame of 256 tokens 32.8 and 35.3 us, four 576-token images 37.8
// and 40.3, one sample of 2880 tokens 47.2 and 49.0).
struct KsChoice { int waves, split; };
#define DART_KS_SHAPES(X_)                                                                   \
  X_(3, 1) X_(4, 1) X_(5, 1) X_(6, 1) X_(8, 1) X_(9, 1) X_(10, 1) X_(11, 1) X_(12, 1)        \
  X_(4, 2) X_(6, 2) X_(8, 2) X_(12, 2) X_(6, 3) X_(9, 3) X_(12, 3)                          \
  X_(8, 4) X_(12, 4) X_(16, 4) X_(8, 8)
constexpr KsChoice kKsShapes[] = {
#define DART_KS_ENTRY(W, KS) {W, KS},
    DART_KS_SHAPES(DART_KS_ENTRY)
#undef DART_KS_ENTRY
};
constexpr size_t kKsLdsLimit = 150 * 1024;  // of the 160 KB of a compute unit

// first_read: the score pass is the first pass of the call over X (pivots given or drawn, a
// separate criterion tensor, the stage entry point), so no norm pass has left the rows in the
// memory-side cache.
KsChoice choose_score_tiles(const Geo& g, int units, bool first_read) {
  const int NB = g.Ppad / 16;
  // Thousands of tiles spread evenly by themselves, and short ones end together.  Packed batches: from
  // 131 000 rows on (whole call with 64-row tiles and with the model's, rows of 1024 to 8192: sixteen
  // samples, 131 000 rows, 150 and 155 us to 835 and 862; 200 of 800 tokens 194 and 197 to 990 and 1031;
  // 32 samples, 290 000 rows of 3584, 793 and 804).  Dense ones, whose tiles the model can make fill the
  // units, from 197 000 (64 of 4096 tokens 155.6 and 156.5 to 619 and 626, 230 of 1500 520 and 532 at
  // 2048; at most 0.7 % behind, on 512 of 576); below, the model's are up to 2.5 % ahead (48 of 2880 335
  // and 341 at 3584, 738 and 756 at 8192).
  if (NB == 1 && g.total_N >= (g.cu ? 512L : 768L) * units) return {4, 1};
  const double rowbytes = (double)g.D * 2;
  const int chunks = (g.D + kKsCH - 1) / kKsCH;
  struct Cost {
    double t, rows_busiest;
    bool fits;
  };
  auto cost = [&](const KsChoice& c) -> Cost {
    const int R = 16 * c.waves / c.split;
    const size_t lds = ksplit_lds_bytes(NB, c.split, c.waves);
    if (lds > kKsLdsLimit) return {1e30, 0.0, false};
    const double tiles = g.cu == nullptr ? (double)g.B * ((g.N + R - 1) / R)
                                         : (double)g.total_N / R + 0.5 * g.B;
    const double per_unit = std::ceil(tiles / units);
    const double rows_busiest = per_unit * R;
    const double rows_avg = (double)g.total_N / units;
    const double weight = 1.0 + 0.2 * NB * 16 / R;  // pivot chunks come from L2
    double t = g.total_N * rowbytes * weight / 6.0e12;
    if (rows_busiest > rows_avg) t += (rows_busiest - rows_avg) * rowbytes * weight / 48e9;
    const int resident = (int)std::max<size_t>(1, std::min<size_t>(kKsLdsLimit / lds, 16 / c.waves));
    const double chain = std::ceil(per_unit / resident) * ((chunks + c.split - 1) / c.split) * 0.55e-6 + 4e-6;
    t = std::max(t, chain);
    t += 1e-9 * (256 - R) / 256;  // ties: the taller tile (less pivot traffic)
    return {t, rows_busiest, true};
  };
  KsChoice best = {4, 1};
  double best_t = 1e30;
  for (const KsChoice& c : kKsShapes) {
    const Cost k = cost(c);
    if (k.fits && k.t < best_t) {
      best_t = k.t;
      best = c;
    }
  }
  // What the model does not see, measured with every shape forced in turn (score pass by the
  // launch's own events): where a wave's chain of chunks matters, four groups of waves per
  // tile beat two or three of the same tile height (32 rows: 8 waves in 4 groups 15.9 us
  // against 17.4 for 6 in 3 on 32 samples of 256 tokens; 48 rows: 12 in 4 groups 15.2 against
  // 17.2 for 6 in 2 on sixteen 576-token images, 22.1 against 25.2 at a hidden size of 5120; whole call
  // with the present score pass 55.8 and 57.4, 67.8 and 69.8) ...
  const int R_best = 16 * best.waves / best.split;
  if (best.split >= 2 && best.split < 4 && (R_best == 32 || R_best == 48)) {
    const KsChoice four = {R_best / 4, 4};
    if (cost(four).fits) return four;
  }
  // ... a unit that gets one tile of at most 5 waves has too few loads in flight: two groups on a tile
  // of about the same height (score pass of eight samples of 2100 tokens in tiles of 96 rows of two groups
  // and of 80 rows of one: 20.7 and 21.6 us, with 32 pivots 21.6 and 23.8, with 64 31.5 and 38.1, on a
  // first read 30.6 and 32.5; eight of 2560, whose 80-row tiles fill the units: 24.3 and 23.9, 23.3 and
  // 24.8, 32.5 and 38.5; eight of 2048, 64 rows: 19.9 and 21.4; whole call on eight spans, 15249 rows of
  // 3584: 105.7 -> 99.7) ...
  // On a first read the 96-row ones stay (eight samples of 2100 and 2560 tokens with rows of 2048: 15.7 and
  // 16.8 us against 18.3 and 19.5 in one group, 18.6 and 19.3 in four; of 8192 57.9 and 60.2, 63.6 and
  // 65.4, 66.5 and 62.4; of 4096 as fast as four but for sixteen of 1280, 36.7 and 31.0) ...
  KsChoice pick = best;
  if (best.split == 1 && best.waves <= 5 && cost(best).rows_busiest == R_best) {
    const KsChoice two = {best.waves == 3 ? 6 : best.waves == 4 ? 8 : 12, 2};
    if (cost(two).fits) pick = two;
    if (best.waves == 5) return pick;
  }
  // ... and the others give way to four groups on small dense batches as
  // long as no compute unit gets more rows: up to 96 (score pass of eight samples of 2048 tokens, 32-row
  // tiles of four groups and 64-row tiles of two: 23.7 and 28.4 us, rows of 8192 53.1 and 54.4; of 3000
  // tokens 32.6 and 34.5 in one group, rows of 8192 64.6 and 72.5; the headline batch 32.8-34.4 and 39.1),
  // and up to 128 where the tiles leave no unit idle and rows are long (eight of 4096 43.8 and 53.1, rows of
  // 8192 96 and 106; sixteen of 2000 42.3 and 43.3, rows of 8192 95 and 103, but of 2048 25.2 and 23.0, of 1024
  // 17.0 and 13.7; eight of 3600 40.8 and 37.6, five of 5000 36.2 and 32.2).  With 32 pivots fewer groups
  // stay ahead: 31.4 and 28.8 on eight of 2048, 59.5 and 45.6 on eight of 2880.
  if (first_read && best.split == 1 && NB == 1 && g.cu == nullptr) {
    const Cost picked = cost(pick);
    const bool full = (double)g.total_N / units >= 0.95 * picked.rows_busiest && chunks >= 32;
    if (picked.rows_busiest <= (full ? 128 : 96)) {
      // (of the two, the one that loads the busiest unit less; equal: the 32-row tiles, two
      // workgroups of which share a unit: 34.7 against 35.5-36.3 us on the headline batch)
      double alt_rows = picked.rows_busiest + 1;
      for (const KsChoice& c : {KsChoice{8, 4}, KsChoice{12, 4}}) {
        const Cost k = cost(c);
        if (k.fits && k.rows_busiest <= picked.rows_busiest && k.rows_busiest < alt_rows) {
          alt_rows = k.rows_busiest;
          pick = c;
        }
      }
    }
  }
  return pick;
}

// Tiles of the fp32 score kernels: rows 2 (k_scores_f32_rows), 4 (k_scores_f32_t4, 4 * groups pivots
// each) or 16 to 32 (k_scores_f32_t16).  All run at the speed of the compute unit that takes in the
// most, token rows and the pivots that every tile reads again (ragged batches: half a tile is lost per
// sample): the cheapest in rounds of the chip times rows per workgroup, weighted by how fast a kernel
// takes rows in (its score pass on 40 to 9216 rows of 512 to 8192, 1 to 64 pivots: the choice is within
// 1 % of the best on average; k_scores_f32_rows pays from rows of 12 KiB on).  Heights on 5776 rows of
// 2048 with 16 pivots: 16, 20, 24, 28, 32 rows per tile take 20.0, 28.0, 17.4, 17.7, 18.8 us; above 48
// pivots a second block of rows does not fit the registers: 16 rows.
struct F32Tile { int rows, groups; };
F32Tile f32_tile(const Geo& g, int units) {
  auto tiles = [&](int rows) {
    return g.cu == nullptr ? (long)g.B * ((g.N + rows - 1) / rows)
                           : (long)g.total_N / rows + (g.B + 1) / 2;
  };
  auto rounds = [&](long blocks) { return (double)((blocks + units - 1) / units); };
  F32Tile best = {16, 0};
  double best_cost = 1e300;
  auto consider = [&](int rows, int groups, double cost) {
    if (cost >= best_cost) return;
    best = {rows, groups};
    best_cost = cost;
  };
  for (int rows = 16; rows <= (g.P > 48 ? 16 : 32); rows += 4)
    consider(rows, 0, rounds(tiles(rows)) * (rows + g.P) * (g.P <= 16 ? 1.0 : 1.1));
  for (int groups = 1; groups <= 4; groups *= 2) {
    const int per = 4 * groups;
    consider(4, groups, rounds(tiles(4) * ((g.P + per - 1) / per)) * (4 + std::min(per, g.P)) *
                            (groups == 1 ? 1.0 : groups == 2 ? 1.3 : 1.5));
  }
  if (g.D > 3072 && g.P <= 24 && g.total_N <= 8L * units)
    consider(2, 0, rounds(tiles(2)) * ((g.P + kF32Piv - 1) / kF32Piv) * (kF32Rows + kF32Piv) *
                       (g.D > 4096 ? 0.65 : g.P <= 8 ? 0.6 : 0.9));
  return best;
}

// Upper bound of the number of score tiles for the tile height in p.g.tile_rows.
void size_score_tiles(Plan& p) {
  if (p.g.cu == nullptr)
    p.tiles_bound = p.g.B * ((p.g.N + p.g.tile_rows - 1) / p.g.tile_rows);
  else
    p.tiles_bound = (int)(p.g.total_N / p.g.tile_rows) + p.g.B;
}

// DART_SCORE_TILE="W,KS" in the environment names the shape instead (for tuning, and for the
// tests that run every instantiated shape); a value that is not one of the shapes above, or
// does not fit the LDS with this many pivots, is an error of the call.
dart_status plan_score_tiles(Plan& p, bool first_read) {
  KsChoice c = choose_score_tiles(p.g, compute_units(), first_read);
  if (const char* v = std::getenv("DART_SCORE_TILE")) {
    int w = 0, ks = 0;
    bool known = false;
    if (std::sscanf(v, "%d,%d", &w, &ks) == 2)
      for (const KsChoice& k : kKsShapes) known = known || (k.waves == w && k.split == ks);
    if (!known || ksplit_lds_bytes(p.g.Ppad / 16, ks, w) > kKsLdsLimit) return DART_ERR_SHAPE;
    c = {w, ks};
  }
  p.ks_waves = c.waves;
  p.ks_split = c.split;
  p.g.tile_rows = 16 * c.waves / c.split;
  size_score_tiles(p);
  return DART_OK;
}

// An entry point whose score pass is the first pass over X plans its tiles again (make_plan
// assumes a norm pass over X before it).
dart_status replan_first_read(Plan& p) {
  return p.g.dtype == kBF16 ? plan_score_tiles(p, true) : DART_OK;
}

dart_status make_plan(const dart_desc* d, Plan& p) {
  if (!d) return DART_ERR_NULL;
  if (d->dtype != DART_F32 && d->dtype != DART_BF16) return DART_ERR_DTYPE;
  if (d->pivot_mode != DART_PIVOT_MAX_L1 && d->pivot_mode != DART_PIVOT_MIN_L1 &&
      d->pivot_mode != DART_PIVOT_GIVEN && d->pivot_mode != DART_PIVOT_RANDOM)
    return DART_ERR_DTYPE;
  if (d->B < 0 || d->B > kMaxB || d->D <= 0 || d->D > 65536 || d->P < 1 || d->P > kMaxP || d->ld < d->D ||
      d->ld > kMaxLd || d->score_mode < 0 || d->score_mode > 2 || d->P_ext < 0 || d->P_ext > d->P)
    return DART_ERR_SHAPE;
  const int Pin = d->P - d->P_ext;  // pivots that are tokens of the sample
  const bool ragged = d->cu_seqlens != nullptr;
  long total;
  int maxn;
  if (!ragged) {
    if (d->N < 0 || d->N > kMaxN) return DART_ERR_SHAPE;
    total = (long)d->B * d->N;
    if (d->total_N != 0 && d->total_N != total) return DART_ERR_SHAPE;
    maxn = d->N;
  } else {
    if (d->total_N < 0 || d->max_N < 1 || d->max_N > kMaxN) return DART_ERR_SHAPE;
    total = d->total_N;
    maxn = d->max_N;
  }
  if (total > (1L << 27)) return DART_ERR_SHAPE;
  if (d->span_start) {  // spans of a larger tensor: packed lengths required, X_rows bounds them
    if (!ragged) return DART_ERR_NULL;
    if (d->X_rows < total || d->X_rows > (1 << 30)) return DART_ERR_SHAPE;
  }
  if (d->K < 0) return DART_ERR_BUDGET;
  if (d->K == 0 && (d->keep_den <= 0 || d->keep_num < 0 || d->keep_num > d->keep_den))
    return DART_ERR_BUDGET;
  int K = d->K;
  if (!ragged) {
    if (K == 0) K = (int)(((long)d->N * d->keep_num) / d->keep_den);
    if (d->B > 0 && (Pin > d->N || K < Pin || K > d->N)) return DART_ERR_BUDGET;
  } else if (K > 0 && (K < Pin || K > maxn)) {
    return DART_ERR_BUDGET;
  }
  const int esz = d->dtype == DART_BF16 ? 2 : 4;
  if (((long)d->ld * esz) % 16 != 0 || ((long)d->D * esz) % 16 != 0) return DART_ERR_ALIGN;
  if (d->P_ext > 0) {
    if (!d->ext_pivots) return DART_ERR_NULL;
    if (d->ext_ld < d->D || d->ext_ld > kMaxLd) return DART_ERR_SHAPE;
    if ((reinterpret_cast<uintptr_t>(d->ext_pivots) & 15u) != 0 || ((long)d->ext_ld * esz) % 16 != 0)
      return DART_ERR_ALIGN;
  }

  Geo& g = p.g;
  g.B = d->B;
  g.D = d->D;
  g.P = d->P;
  g.Ppad = (d->P + 15) / 16 * 16;
  g.N = ragged ? 0 : d->N;
  g.total_N = (int)total;
  g.max_N = maxn;
  g.K = ragged ? d->K : K;
  g.keep_num = d->keep_num;
  g.keep_den = d->keep_den > 0 ? d->keep_den : 1;
  g.dtype = d->dtype;
  g.mode = d->pivot_mode;
  p.seed = d->seed;
  g.score_mode = d->score_mode;
  g.ld = d->ld;
  g.cu = d->cu_seqlens;
  g.cu_keep = nullptr;
  g.tile_start = nullptr;
  g.by_size = nullptr;
  g.Pe = d->P_ext;
  g.Pin = Pin;
  g.lde = d->P_ext > 0 ? d->ext_ld : 0;
  g.E = d->P_ext > 0 ? d->ext_pivots : nullptr;
  g.span = d->span_start;
  g.x_rows = d->span_start ? d->X_rows : (int)total;
  // score tiles: the kernel and height (fp32) or the shape (bf16) chosen for this batch
  p.ks_waves = p.ks_split = p.f32_groups = 0;
  if (d->dtype == DART_BF16) {
    // (pivots given, drawn or all from outside: no norm pass reads X before the score pass)
    const dart_status ts = plan_score_tiles(p, d->pivot_mode == DART_PIVOT_GIVEN ||
                                                   d->pivot_mode == DART_PIVOT_RANDOM || Pin == 0);
    if (ts != DART_OK) return ts;
  } else {
    const F32Tile t = f32_tile(g, compute_units());
    g.tile_rows = t.rows;
    p.f32_groups = t.groups;
  }
  p.esz = esz;
  if (!ragged) {
    p.keep_rows_bound = (long)d->B * K;
  } else {
    p.keep_rows_bound = d->K > 0 ? (long)d->B * d->K
                                 : (long)(((__int128)total * d->keep_num) / g.keep_den);
    if (p.keep_rows_bound > total) p.keep_rows_bound = total;
  }
  size_score_tiles(p);
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o += up(bytes); return at; };
  p.o_status = take(kAlign);
  p.o_cu_keep = take(sizeof(int) * ((size_t)d->B + 1));
  p.o_tile_start = take(sizeof(int) * ((size_t)d->B + 1));
  p.o_l1 = take(sizeof(float) * (size_t)total);
  p.o_piv = take(sizeof(int) * (size_t)d->B * d->P);
  p.o_pl2 = take(sizeof(double) * (size_t)d->B * g.Ppad);
  p.o_S = take(sizeof(float) * (size_t)total * d->P);
  p.o_lists = take(sizeof(unsigned long long) * (size_t)total * d->P);
  p.o_scr_f64 = take(sizeof(double) * 2 * (size_t)total);
  p.o_l2 = take(sizeof(double) * (size_t)total);
  // one-launch path: bf16, pivots chosen among the tokens, the staged rule, packed samples
  p.fusable = d->dtype == DART_BF16 && d->pivot_mode != DART_PIVOT_GIVEN &&
              d->pivot_mode != DART_PIVOT_RANDOM && d->P_ext == 0 &&
              d->score_mode == 0 && d->span_start == nullptr && d->B <= kFuMaxB;
  if (d->B <= kFuMaxB) {  // (the same workspace size whatever the modes)
    p.o_sync = take(sizeof(int) * (size_t)fused_sync_ints(d->B, d->P));
    p.o_nstart = take(sizeof(int) * ((size_t)d->B + 1));
    p.o_sstart = take(sizeof(int) * ((size_t)d->B + 1));
    p.o_gstart = take(sizeof(int) * ((size_t)d->B + 1));
  } else {
    p.o_sync = p.o_nstart = p.o_sstart = p.o_gstart = o;
  }
  p.o_by_size = take(sizeof(int) * kMaxBySize);
  p.norms_given = false;
  p.total = o;
  return DART_OK;
}

inline bool misaligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

dart_status check_ws(const Plan& p, const void* ws, size_t ws_bytes) {
  if (!ws || (reinterpret_cast<uintptr_t>(ws) % kAlign) != 0 || ws_bytes < p.total)
    return DART_ERR_WORKSPACE;
  return DART_OK;
}

template <typename T>
inline T* at(void* ws, size_t off) {
  return reinterpret_cast<T*>(static_cast<unsigned char*>(ws) + off);
}

#define DART_LAUNCH_CHECK()                              \
  do {                                                   \
    if (hipGetLastError() != hipSuccess) return DART_ERR_HIP; \
  } while (0)

// Stage events of dart_reduce_profiled.  While they are set, every kernel this thread launches
// stamps them with its own begin and end (the start/stop events of hipExtLaunchKernel: the
// times are the dispatch's, and no marker packet goes between the kernels, so a stage's
// elapsed time is what a kernel trace shows for it); the first kernel of a stage takes the
// start event, every kernel of the stage the stop event (the last one's time stays).
struct StageEvents {
  hipEvent_t start = nullptr, stop = nullptr;
};
thread_local StageEvents t_stage;

#define DART_LAUNCH(kernel, grid, block, shmem, st, ...)                                        \
  do {                                                                                          \
    if (t_stage.stop != nullptr) {                                                              \
      hipExtLaunchKernelGGL(kernel, grid, block, shmem, st, t_stage.start, t_stage.stop, 0,     \
                            __VA_ARGS__);                                                       \
      t_stage.start = nullptr;                                                                  \
    } else {                                                                                    \
      hipLaunchKernelGGL(kernel, grid, block, shmem, st, __VA_ARGS__);                          \
    }                                                                                           \
  } while (0)

#define DART_TRY(expr)                    \
  do {                                    \
    dart_status _s = (expr);              \
    if (_s != DART_OK) return _s;         \
  } while (0)

// Points g at the ragged offsets in the workspace (no-op for dense batches); the caller launches
// what fills them.
PrepareArgs prepare_args(Plan& p, void* ws) {
  PrepareArgs a = {};
  if (p.g.cu == nullptr) return a;
  a.cu_keep = at<int>(ws, p.o_cu_keep);
  a.tile_start = at<int>(ws, p.o_tile_start);
  a.status = at<int>(ws, p.o_status);
  // (only where the ordering kernel's B*P workgroups, one per compute unit, need several rounds)
  a.by_size = p.g.B <= kMaxBySize && (long)p.g.B * p.g.P > compute_units()
                  ? at<int>(ws, p.o_by_size) : nullptr;
  p.g.cu_keep = a.cu_keep;
  p.g.tile_start = a.tile_start;
  p.g.by_size = a.by_size;
  return a;
}

// Fills the ragged offsets (no-op for dense batches).  seq_cu, seq_cu_out: see PrepareArgs.
dart_status launch_prepare(Plan& p, void* ws, hipStream_t st, const int* seq_cu = nullptr,
                           int* seq_cu_out = nullptr) {
  if (p.g.cu == nullptr) return DART_OK;
  PrepareArgs a = prepare_args(p, ws);
  a.seq_cu = seq_cu;
  a.seq_cu_out = seq_cu_out;
  DART_LAUNCH(k_prepare, dim3(1), dim3(1024), 0, st, p.g, a);
  DART_LAUNCH_CHECK();
  return DART_OK;
}

// keep_cached: the rows will be read again soon (they are the hidden states themselves).
// Ragged batches: also fills the ragged offsets, by a block of the same launch for up to
// kPrepareInPass samples: as a launch of its own that takes 4-5 us first, however few they are, but a
// block of the pass is 256 threads and takes about 0.5 us per 256 samples, which with many short
// samples is longer than the rest of the pass (norms and selection of samples of at most 8 tokens of
// 64 elements, in the pass and with the launch: 1000 samples 13.4 and 16.3 us, 4096 34.3 and 34.5, 8192
// 60.6 and 58.2, 65536 485 and 400).
constexpr int kPrepareInPass = 2048;
// Rows of at most 64 pieces: eight to a wave (156 000 rows of 512 bytes: 40 us
// with one, 17).
constexpr long kShortRowBytes = kWave * 16;
dart_status launch_row_l1(Plan& p, const void* C, int Dc, long ldc, float* l1, bool keep_cached,
                          void* ws, hipStream_t st, double* l2sq = nullptr) {
  double* l1d = at<double>(ws, p.o_scr_f64);
  const int rows = p.g.total_N;
  if (rows == 0) return launch_prepare(p, ws, st);
  const bool fill = p.g.cu != nullptr && p.g.B <= kPrepareInPass;
  if (!fill) DART_TRY(launch_prepare(p, ws, st));
  const PrepareArgs prep = prepare_args(p, ws);
  if (l2sq == nullptr && p.g.span == nullptr && (long)Dc * p.esz <= kShortRowBytes) {
    const dim3 grid((unsigned)round_up8((rows + 31) / 32) + (fill ? kXcds : 0));
#define DART_LAUNCH_SHORT(DT, PREP)                                                              \
  DART_LAUNCH((k_short_row_l1<DT, 8, PREP>), grid, dim3(256), 0, st, C, Dc, ldc, rows, l1, l1d,  \
              p.g, prep)
    if (p.g.dtype == kBF16) {
      if (fill) DART_LAUNCH_SHORT(kBF16, true); else DART_LAUNCH_SHORT(kBF16, false);
    } else {
      if (fill) DART_LAUNCH_SHORT(kF32, true); else DART_LAUNCH_SHORT(kF32, false);
    }
#undef DART_LAUNCH_SHORT
    DART_LAUNCH_CHECK();
    return DART_OK;
  }
  const int blocks = (int)round_up8((rows + 3) / 4) + (fill ? kXcds : 0);
  // The 256 MB memory-side cache serves the score kernel's second pass if this pass leaves
  // the rows there: measured 31 instead of 38 us on that kernel for 0.7 us more on this one
  // at 189 MB; at 264 MB this pass loses 7 us and that one gains 0.7; a loss for matrices
  // that cannot fit.
  // With spans the caller moves whole sequences afterwards, which sweeps that cache anyway:
  // measured slower with ordinary loads there.
  const bool keep = keep_cached && (double)rows * ldc * p.esz <= 224e6;
#define DART_LAUNCH_L1_AS(DT, KEEP, SPAN, L2SQ)                                                  \
  do {                                                                                           \
    if (fill)                                                                                    \
      DART_LAUNCH((k_row_l1<DT, KEEP, SPAN, L2SQ, true>), dim3(blocks), dim3(256), 0, st,        \
                  C, Dc, ldc, rows, l1, l1d, p.g, l2sq, prep);                                   \
    else                                                                                         \
      DART_LAUNCH((k_row_l1<DT, KEEP, SPAN, L2SQ, false>), dim3(blocks), dim3(256), 0, st,       \
                  C, Dc, ldc, rows, l1, l1d, p.g, l2sq, prep);                                   \
  } while (0)
#define DART_LAUNCH_L1(DT)                                                                       \
  do {                                                                                           \
    if (l2sq && p.g.span) DART_LAUNCH_L1_AS(DT, false, true, true);                              \
    else if (l2sq && keep) DART_LAUNCH_L1_AS(DT, true, false, true);                             \
    else if (l2sq) DART_LAUNCH_L1_AS(DT, false, false, true);                                    \
    else if (p.g.span) DART_LAUNCH_L1_AS(DT, false, true, false);                                \
    else if (keep) DART_LAUNCH_L1_AS(DT, true, false, false);                                    \
    else DART_LAUNCH_L1_AS(DT, false, false, false);                                             \
  } while (0)
  if (p.g.dtype == kBF16) DART_LAUNCH_L1(kBF16); else DART_LAUNCH_L1(kF32);
#undef DART_LAUNCH_L1
#undef DART_LAUNCH_L1_AS
  DART_LAUNCH_CHECK();
  return DART_OK;
}

// Values a thread of the selection kernels keeps in registers: 1024 threads times this many
// cover the longest sample (see k_select.hpp); instantiated for 1, 2, 3, 4, 6, 8, 10, 12, 16.
int values_per_thread(int max_n) {
  const int need = (max_n + 1023) / 1024;
  for (int per : {1, 2, 3, 4, 6, 8, 10, 12, 16})
    if (per >= need) return per;
  return 16;
}
#define DART_FOR_VALUES_PER_THREAD(per, LAUNCH)                                                  \
  switch (per) {                                                                                 \
    case 1: LAUNCH(1); break;                                                                    \
    case 2: LAUNCH(2); break;                                                                    \
    case 3: LAUNCH(3); break;                                                                    \
    case 4: LAUNCH(4); break;                                                                    \
    case 6: LAUNCH(6); break;                                                                    \
    case 8: LAUNCH(8); break;                                                                    \
    case 10: LAUNCH(10); break;                                                                  \
    case 12: LAUNCH(12); break;                                                                  \
    default: LAUNCH(16); break;                                                                  \
  }

// l1_rel_err < 0: the norms are the norm pass's own (rounded fp64 norms, which lie in the scratch
// area); otherwise the caller's, good to that relative error.  l2sq: the squared norms of the hidden
// states' rows if the norm pass left them.  pl2: receives those of the pivots, or nullptr.
dart_status launch_select_pivots(const Plan& p, const void* X, const void* C, int Dc, long ldc,
                                 const float* l1, const double* l2sq, int* piv, double* pl2, void* ws,
                                 hipStream_t st, double l1_rel_err = -1.0) {
  // (the bound plus the rounding of the threshold arithmetic itself, so that exact norms rounded
  // to fp32 still hold every exact pivot)
  const float tau = (float)(std::max(l1_rel_err, 0.0) + 1.2e-7);
  double* l1d = at<double>(ws, p.o_scr_f64);
  // 1024 threads: a 256-thread variant measured slower even for short samples
  // (up to 4096 tokens: samples longer than that by the hundred take milliseconds elsewhere)
  const bool two = p.g.B > compute_units();
#define DART_LAUNCH_PIVOTS_AS(DT, PER, EXACT, TWO)                                               \
  DART_LAUNCH((k_select_pivots<DT, PER, EXACT, TWO>), dim3(p.g.B), dim3(1024), 0, st, p.g, X, C, \
              Dc, ldc, l1, piv, pl2, l1d, l2sq, tau)
#define DART_LAUNCH_PIVOTS_DT(DT, PER)                                                           \
  do {                                                                                           \
    if (l1_rel_err >= 0) DART_LAUNCH_PIVOTS_AS(DT, PER, false, false);                           \
    else if (two && PER <= 4) DART_LAUNCH_PIVOTS_AS(DT, PER, true, (PER <= 4));                  \
    else DART_LAUNCH_PIVOTS_AS(DT, PER, true, false);                                            \
  } while (0)
#define DART_LAUNCH_PIVOTS(PER)                                                                  \
  do {                                                                                           \
    if (p.g.dtype == kBF16) DART_LAUNCH_PIVOTS_DT(kBF16, PER);                                   \
    else DART_LAUNCH_PIVOTS_DT(kF32, PER);                                                       \
  } while (0)
  DART_FOR_VALUES_PER_THREAD(values_per_thread(p.g.max_N), DART_LAUNCH_PIVOTS);
#undef DART_LAUNCH_PIVOTS
#undef DART_LAUNCH_PIVOTS_DT
#undef DART_LAUNCH_PIVOTS_AS
  DART_LAUNCH_CHECK();
  return DART_OK;
}

// Norms of all pivots; piv_mark (optional) receives the marks of the pivots from outside the samples.
dart_status launch_pivot_norms(const Plan& p, const void* X, const int* piv, int* piv_mark, void* ws,
                               hipStream_t st) {
  double* pl2 = at<double>(ws, p.o_pl2);
  if (p.g.dtype == kBF16)
    DART_LAUNCH((k_pivot_norms<kBF16>), dim3(p.g.B), dim3(1024), 0, st, p.g, X, piv, pl2, piv_mark);
  else
    DART_LAUNCH((k_pivot_norms<kF32>), dim3(p.g.B), dim3(1024), 0, st, p.g, X, piv, pl2, piv_mark);
  DART_LAUNCH_CHECK();
  return DART_OK;
}

// The pivots of DART_PIVOT_RANDOM, drawn on the device (the first Pin entries of every sample).
// DART_RANDOM_DRAW_LIMIT=n in the environment lowers the rule's limit of 4096 draws per sample
// (0..4096; for the test of the fill that follows the last draw, which no input reaches).
dart_status launch_random_pivots(const Plan& p, int* piv, hipStream_t st) {
  if (p.g.Pin == 0) return DART_OK;
  int limit = kRandomDraws;
  if (const char* v = std::getenv("DART_RANDOM_DRAW_LIMIT")) {
    const int n = std::atoi(v);
    if (n < 0 || n > kRandomDraws) return DART_ERR_SHAPE;
    limit = n;
  }
  DART_LAUNCH(k_random_pivots, dim3(p.g.B), dim3(64), 0, st, p.g, p.seed, limit, piv);
  DART_LAUNCH_CHECK();
  return DART_OK;
}

// Leaves the pivot flag of dart_device_status defined for a DART_PIVOT_GIVEN descriptor: the
// list the entry point reads is validated, or the flag is cleared if it reads none.
dart_status launch_given_status(const Plan& p, const int* piv, void* ws, hipStream_t st) {
  if (p.g.mode != kGiven) return DART_OK;
  if (piv)
    DART_LAUNCH(k_check_pivots, dim3(1), dim3(1024), 0, st, p.g, piv,
                at<int>(ws, p.o_status));
  else
    DART_LAUNCH(k_clear_pivot_status, dim3(1), dim3(1), 0, st, at<int>(ws, p.o_status));
  DART_LAUNCH_CHECK();
  return DART_OK;
}

template <int NB, bool TAIL, bool XN>
dart_status launch_scores_ksplit_nb(const Plan& p, const void* X, const int* piv,
                                    const double* pl2, const double* l2sq, float* S,
                                    hipStream_t st) {
  const dim3 grid((unsigned)round_up8(p.tiles_bound)), block(64 * p.ks_waves);
#define DART_KS_LAUNCH(W, KS)                                                                   \
  if (p.ks_waves == W && p.ks_split == KS) {                                                    \
    if constexpr (ksplit_lds_bytes(NB, KS, W) <= kKsLdsLimit) {                                 \
      DART_LAUNCH((k_scores_ksplit<NB, KS, W, TAIL, XN>), grid, block, 0, st, p.g, X,           \
                  piv, pl2, l2sq, S);                                                           \
      DART_LAUNCH_CHECK();                                                                      \
      return DART_OK;                                                                           \
    }                                                                                           \
  }
  DART_KS_SHAPES(DART_KS_LAUNCH)
#undef DART_KS_LAUNCH
  return DART_ERR_SHAPE;
}

template <int NB>
dart_status launch_scores_ksplit_tx(const Plan& p, const void* X, const int* piv,
                                    const double* pl2, const double* l2sq, float* S,
                                    hipStream_t st) {
  const bool tail = p.g.D % kKsCH != 0;
  if (l2sq)
    return tail ? launch_scores_ksplit_nb<NB, true, true>(p, X, piv, pl2, l2sq, S, st)
                : launch_scores_ksplit_nb<NB, false, true>(p, X, piv, pl2, l2sq, S, st);
  return tail ? launch_scores_ksplit_nb<NB, true, false>(p, X, piv, pl2, l2sq, S, st)
              : launch_scores_ksplit_nb<NB, false, false>(p, X, piv, pl2, l2sq, S, st);
}

// l2sq: the squared token norms if this call's norm pass left them (else the score kernel
// takes them from its own Gram products).
dart_status launch_scores(const Plan& p, const void* X, const int* piv, float* S, void* ws,
                          hipStream_t st) {
  if (p.tiles_bound == 0) return DART_OK;
  const double* pl2 = at<double>(ws, p.o_pl2);
  const double* l2sq = p.norms_given ? at<double>(ws, p.o_l2) : nullptr;
  if (p.g.dtype == kF32) {
#define DART_LAUNCH_F32(KERNEL, PIVOTS, THREADS)                                                 \
  DART_LAUNCH((KERNEL), dim3(p.tiles_bound, (p.g.P + (PIVOTS) - 1) / (PIVOTS)), dim3(THREADS), 0, \
              st, p.g, X, piv, pl2, S)
    constexpr int threads = kF32Waves * 64;
    if (p.g.tile_rows == kF32Rows) {
      DART_LAUNCH_F32(k_scores_f32_rows, kMaxP, 256);
    } else if (p.g.tile_rows == 4) {
      switch (p.f32_groups) {
        case 1: DART_LAUNCH_F32(k_scores_f32_t4<1>, 4, threads); break;
        case 2: DART_LAUNCH_F32(k_scores_f32_t4<2>, 8, threads); break;
        default: DART_LAUNCH_F32(k_scores_f32_t4<4>, 16, threads); break;
      }
    } else {
#define DART_LAUNCH_F32_NB(NB)                                                                   \
  do {                                                                                           \
    if (p.g.tile_rows == 16) DART_LAUNCH_F32((k_scores_f32_t16<NB, 1>), kMaxP, threads);         \
    else DART_LAUNCH_F32((k_scores_f32_t16<NB, 2>), kMaxP, threads);                             \
  } while (0)
      switch (p.g.Ppad / 16) {
        case 1: DART_LAUNCH_F32_NB(1); break;
        case 2: DART_LAUNCH_F32_NB(2); break;
        case 3: DART_LAUNCH_F32_NB(3); break;
        default: DART_LAUNCH_F32((k_scores_f32_t16<4, 1>), kMaxP, threads); break;  // (f32_tile)
      }
#undef DART_LAUNCH_F32_NB
    }
#undef DART_LAUNCH_F32
    DART_LAUNCH_CHECK();
    return DART_OK;
  }
  switch (p.g.Ppad / 16) {
    case 1: return launch_scores_ksplit_tx<1>(p, X, piv, pl2, l2sq, S, st);
    case 2: return launch_scores_ksplit_tx<2>(p, X, piv, pl2, l2sq, S, st);
    case 3: return launch_scores_ksplit_tx<3>(p, X, piv, pl2, l2sq, S, st);
    default: return launch_scores_ksplit_tx<4>(p, X, piv, pl2, l2sq, S, st);
  }
}

dart_status launch_order(const Plan& p, const float* S, void* ws, hipStream_t st) {
  if (p.g.score_mode != 0) return DART_OK;  // the single-threshold rule orders nothing per pivot
  unsigned long long* lists = at<unsigned long long>(ws, p.o_lists);
  // 1024 threads: a 256-thread variant measured slower even for short samples
#define DART_LAUNCH_ORDER(PER)                                                                   \
  DART_LAUNCH((k_order_scores<1024, PER>), dim3(p.g.B * p.g.P), dim3(1024), 0, st, p.g, S,       \
              lists)
  // samples of at most 1024 tokens: 512 threads with two values each (measured on 576-token
  // samples: 8.9 against 9.6 us; pivot selection is slower that way, 3072-token samples too)
  if (p.g.max_N <= 1024)
    DART_LAUNCH((k_order_scores<512, 2>), dim3(p.g.B * p.g.P), dim3(512), 0, st, p.g, S,
                lists);
  else
    DART_FOR_VALUES_PER_THREAD(values_per_thread(p.g.max_N), DART_LAUNCH_ORDER);
#undef DART_LAUNCH_ORDER
  DART_LAUNCH_CHECK();
  return DART_OK;
}

// pivot_norms_ready: this call has left the pivots' fp64 squared norms in the workspace.
dart_status launch_retain(const Plan& p, const float* S, const int* piv, const void* X, int* keep,
                          int* cu_keep, void* ws, hipStream_t st, bool pivot_norms_ready) {
  const double* pl2 = pivot_norms_ready ? at<double>(ws, p.o_pl2) : nullptr;
  const float two_tau = (float)(2.0 * 1.01 * score_abs_bound(p.g.dtype, p.norms_given ? kNormsF64 : kNormsGram));
  const unsigned long long* lists = at<unsigned long long>(ws, p.o_lists);
  double* scr_f64 = at<double>(ws, p.o_scr_f64);
  if (p.g.score_mode != 0) {  // one threshold for all pivots: no stage lists
#define DART_LAUNCH_SINGLE(PER)                                                                  \
  do {                                                                                           \
    if (p.g.dtype == kBF16)                                                                      \
      DART_LAUNCH((k_keep_single<kBF16, PER>), dim3(p.g.B), dim3(1024), 0, st, p.g, S,           \
                  piv, X, keep, cu_keep, scr_f64, two_tau, p.g.score_mode);                      \
    else                                                                                         \
      DART_LAUNCH((k_keep_single<kF32, PER>), dim3(p.g.B), dim3(1024), 0, st, p.g, S,            \
                  piv, X, keep, cu_keep, scr_f64, two_tau, p.g.score_mode);                      \
  } while (0)
    {
      const int per = values_per_thread(p.g.max_N);
      if (per <= 4) DART_LAUNCH_SINGLE(4);
      else if (per <= 8) DART_LAUNCH_SINGLE(8);
      else if (per <= 12) DART_LAUNCH_SINGLE(12);
      else DART_LAUNCH_SINGLE(16);
    }
#undef DART_LAUNCH_SINGLE
    DART_LAUNCH_CHECK();
    return DART_OK;
  }
  // (of the batch's longest sample)
  const int k_big = p.g.K > 0 ? p.g.K : (int)(((long)p.g.max_N * p.g.keep_num) / p.g.keep_den);
  const int quota = (k_big - p.g.Pin) / p.g.P;
  const bool wide = quota >= kWideQuota || (long)quota * p.g.P > kWideSlots;
#define DART_LAUNCH_RETAIN(DT, WIDE)                                                             \
  DART_LAUNCH((k_retain<DT, WIDE>), dim3(p.g.B), dim3(kRetThreads), 0, st, p.g, S, lists, piv, X, \
              keep, cu_keep, scr_f64, two_tau, pl2)
  if (p.g.dtype == kBF16) {
    if (wide) DART_LAUNCH_RETAIN(kBF16, true); else DART_LAUNCH_RETAIN(kBF16, false);
  } else {
    if (wide) DART_LAUNCH_RETAIN(kF32, true); else DART_LAUNCH_RETAIN(kF32, false);
  }
#undef DART_LAUNCH_RETAIN
  DART_LAUNCH_CHECK();
  return DART_OK;
}

dart_status launch_gather(const Plan& p, const void* X, const int64_t* pos, const int* keep,
                          void* Y, int64_t* pos_out, hipStream_t st) {
  if (p.keep_rows_bound == 0) return DART_OK;
  const int blocks = (int)round_up8((p.keep_rows_bound + 3) / 4);
  DART_LAUNCH(k_gather, dim3(blocks), dim3(256), 0, st, p.g, p.esz, X,
              reinterpret_cast<const long long*>(pos), keep, Y,
              reinterpret_cast<long long*>(pos_out));
  DART_LAUNCH_CHECK();
  return DART_OK;
}

// The whole step as one persistent kernel (after a one-workgroup set-up kernel).
dart_status launch_fused(Plan& p, const void* X, const int64_t* pos, void* Y, int64_t* pos_out,
                         int32_t* keep, int32_t* cu_keep, int* piv, float* S, void* ws,
                         hipStream_t st) {
  const int NB = p.g.Ppad / 16;
  const int score_rows = NB <= 2 ? FusedScoreCfg<1>::ROWS : FusedScoreCfg<3>::ROWS;
  int* sync = at<int>(ws, p.o_sync);
  int* nstart = at<int>(ws, p.o_nstart);
  int* sstart = at<int>(ws, p.o_sstart);
  int* gstart = at<int>(ws, p.o_gstart);
  DART_LAUNCH(k_fused_init, dim3(1), dim3(1024), 0, st, p.g, score_rows, Y ? 1 : 0, sync,
              nstart, sstart, gstart, cu_keep, at<int>(ws, p.o_status));
  DART_LAUNCH_CHECK();
  FusedArgs a;
  a.X = X;
  a.pos = reinterpret_cast<const long long*>(pos);
  a.Y = Y;
  a.pos_out = reinterpret_cast<long long*>(pos_out);
  a.keep = keep;
  a.piv = piv;
  a.S = S;
  a.l1 = at<float>(ws, p.o_l1);
  a.l2sq = at<double>(ws, p.o_l2);
  a.pl2 = at<double>(ws, p.o_pl2);
  a.lists = at<unsigned long long>(ws, p.o_lists);
  a.scr = at<double>(ws, p.o_scr_f64);
  a.sync = sync;
  a.norm_start = nstart;
  a.score_start = sstart;
  a.gather_start = gstart;
  a.status = at<int>(ws, p.o_status);
  a.tau_l1 = (float)l1_rel_bound_bf16(p.g.D);
  a.two_tau = (float)(2.0 * 1.01 * score_abs_bound(p.g.dtype, kNormsF32Squares));
  a.keep_cached = (double)p.g.total_N * p.g.ld * p.esz <= 224e6 ? 1 : 0;
  a.spin_limit = 1 << 20;
  const dim3 grid(compute_units()), block(kFuThreads);
  const bool tail = p.g.D % kKsCH != 0;
#define DART_LAUNCH_FUSED(NBV)                                                        \
  do {                                                                                \
    if (tail) DART_LAUNCH((k_fused<NBV, true>), grid, block, 0, st, p.g, a);          \
    else DART_LAUNCH((k_fused<NBV, false>), grid, block, 0, st, p.g, a);              \
  } while (0)
  switch (NB) {
    case 1: DART_LAUNCH_FUSED(1); break;
    case 2: DART_LAUNCH_FUSED(2); break;
    case 3: DART_LAUNCH_FUSED(3); break;
    default: DART_LAUNCH_FUSED(4); break;
  }
#undef DART_LAUNCH_FUSED
  DART_LAUNCH_CHECK();
  return DART_OK;
}

// DART_FUSED=1 in the environment sends dart_reduce through the one-launch kernel where it
// applies (a switch between two complete implementations of the same step; the kernel-per-step
// path is the default because it measured faster on every benchmark shape).
bool fused_enabled() {
  const char* v = std::getenv("DART_FUSED");
  return v && v[0] == '1';
}

dart_status check_crit(const Plan& p, const void* X, const void*& crit, int32_t& crit_D,
                       int64_t& crit_ld) {
  if (!crit) {
    crit = X;
    crit_D = p.g.D;
    crit_ld = p.g.ld;
    return DART_OK;
  }
  if (crit_D <= 0 || crit_D > 65536 || crit_ld < crit_D || crit_ld > kMaxLd) return DART_ERR_SHAPE;
  if (misaligned16(crit) || (crit_ld * p.esz) % 16 != 0 || ((long)crit_D * p.esz) % 16 != 0)
    return DART_ERR_ALIGN;
  return DART_OK;
}

dart_status reduce_impl(const dart_desc* desc, const void* X, const void* crit, int32_t crit_D,
                        int64_t crit_ld, const int64_t* pos, void* Y, int64_t* pos_out,
                        int32_t* keep, int32_t* cu_keep, int32_t* piv_out, float* S_out, void* ws,
                        size_t ws_bytes, void* stream, void* const* events,
                        const float* l1_given = nullptr, double l1_rel_err = 0.0) {
  Plan p;
  DART_TRY(make_plan(desc, p));
  if (l1_given && (p.g.mode == kGiven || p.g.mode == kRandom)) return DART_ERR_DTYPE;
  if (l1_given && !(l1_rel_err >= 0.0 && l1_rel_err <= 0.1)) return DART_ERR_SHAPE;
  if (p.g.B == 0) return DART_OK;
  if (!X || !keep || (Y && (pos != nullptr) != (pos_out != nullptr))) return DART_ERR_NULL;
  if (p.g.mode == kGiven && !piv_out) return DART_ERR_NULL;
  if (misaligned16(X) || (Y && misaligned16(Y))) return DART_ERR_ALIGN;
  // pivots drawn at random: the library writes the list, then the step runs as with a
  // caller's list (no pass over a criterion, no check of a list that is valid by construction)
  const bool random = p.g.mode == kRandom;
  if (random) p.g.mode = kGiven;
  if (p.g.mode == kGiven) crit = nullptr;
  DART_TRY(check_crit(p, X, crit, crit_D, crit_ld));
  // (the first columns of X, or every other row, begin at the same address and are another matrix)
  const bool own_crit = crit == X && crit_D == p.g.D && crit_ld == p.g.ld;
  DART_TRY(check_ws(p, ws, ws_bytes));
  // (the norm pass reads the criterion, not X, or there is none: the caller brought the norms)
  if (!own_crit || l1_given) DART_TRY(replan_first_read(p));
  hipStream_t st = static_cast<hipStream_t>(stream);
  // profiled calls: the kernels launched from here on belong to stage k
  struct StageGuard {
    ~StageGuard() { t_stage = StageEvents{}; }
  } stage_guard;
  auto stage = [&](int k) {
    if (events)
      t_stage = {static_cast<hipEvent_t>(events[2 * k]),
                 static_cast<hipEvent_t>(events[2 * k + 1])};
  };
  int* piv = piv_out ? piv_out : at<int>(ws, p.o_piv);
  float* S = S_out ? S_out : at<float>(ws, p.o_S);
  float* l1 = at<float>(ws, p.o_l1);
  // hidden states as their own criterion: the norm pass also leaves the squared token norms.  Selection takes
  // the pivots' from there instead of summing their rows again (fp32, whole call with and without: one
  // 576-token image 35.2 and 36.7 us, two samples of 9216 with 32 pivots 196 and 204; the fp32 score kernels
  // sum their own), the bf16 score pass saves its Gram products, and the tighter error bound
  // the retained-set kernel 10 % on near-duplicate video frames.  Above 1 GB the norm pass runs at the
  // memory's speed and takes up to 2 % longer with them, the 64-row tiles up to 4 % (100 samples of 2880
  // of 3584, 16 pivots: 766 us with, 756 without; 32 of 8000 of 2048: 392 and 394; with 32 or 48 pivots the
  // call would be 1-3 % faster with them there too: 24 of 9216 of 3584 612 and 620).
  p.norms_given = p.g.mode != kGiven && p.g.Pin > 0 && own_crit &&
                  !l1_given && (double)p.g.total_N * p.g.ld * p.esz <= 1e9;
  // (the one-launch path computes its own norms: not for profiled calls or the caller's norms)
  const bool fused = p.fusable && own_crit && events == nullptr && !l1_given && p.g.total_N > 0 &&
                     fused_enabled();
  // a norm pass fills the ragged offsets on the side (as part of its stage)
  const bool norm_pass = !fused && p.g.mode != kGiven && p.g.Pin > 0 && !l1_given;
  if (!norm_pass) DART_TRY(launch_prepare(p, ws, st));
  stage(0);
  if (fused) return launch_fused(p, X, pos, Y, pos_out, keep, cu_keep, piv, S, ws, st);
  if (p.g.mode == kGiven) {
    // the caller's pivots: check them, compute their norms; no pass over the criterion
    if (random) {
      DART_TRY(launch_random_pivots(p, piv, st));
    } else {
      DART_LAUNCH(k_check_pivots, dim3(1), dim3(1024), 0, st, p.g, piv,
                  at<int>(ws, p.o_status));
      DART_LAUNCH_CHECK();
    }
    stage(1);
    DART_TRY(launch_pivot_norms(p, X, piv, piv, ws, st));
  } else {
    // pivots chosen among the tokens (none if all of them come from outside) ...
    if (norm_pass)
      DART_TRY(launch_row_l1(p, crit, crit_D, crit_ld, l1, own_crit, ws, st,
                             p.norms_given ? at<double>(ws, p.o_l2) : nullptr));
    stage(1);
    // ... with the norms and marks of those from outside
    if (p.g.Pin > 0)
      DART_TRY(launch_select_pivots(p, X, crit, crit_D, crit_ld, l1_given ? l1_given : l1,
                                    p.norms_given ? at<double>(ws, p.o_l2) : nullptr, piv,
                                    at<double>(ws, p.o_pl2), ws, st, l1_given ? l1_rel_err : -1.0));
    else
      DART_TRY(launch_pivot_norms(p, X, piv, piv, ws, st));
  }
  stage(2);
  DART_TRY(launch_scores(p, X, piv, S, ws, st));
  stage(3);
  DART_TRY(launch_order(p, S, ws, st));
  stage(4);
  DART_TRY(launch_retain(p, S, piv, X, keep, cu_keep, ws, st, true));
  stage(5);
  if (Y) DART_TRY(launch_gather(p, X, pos, keep, Y, pos_out, st));  // NULL: the caller compacts
  return DART_OK;
}

// Device address of `scratch` on the current GPU, resolved once per GPU with that GPU current.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

dart_status static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return DART_ERR_HIP;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr)
      return DART_ERR_HIP;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return DART_OK;
}

}  // namespace

extern "C" {

size_t dart_workspace_bytes(const dart_desc* desc) {
  Plan p;
  if (make_plan(desc, p) != DART_OK) return 0;
  return p.total;
}

dart_status dart_score_tile_shape(const dart_desc* desc, int32_t* waves, int32_t* split) {
  if (!waves || !split) return DART_ERR_NULL;
  Plan p;
  DART_TRY(make_plan(desc, p));
  *waves = p.ks_waves;
  *split = p.ks_split;
  return DART_OK;
}

dart_status dart_score_tile_shape_first_read(const dart_desc* desc, int32_t* waves,
                                             int32_t* split) {
  if (!waves || !split) return DART_ERR_NULL;
  Plan p;
  DART_TRY(make_plan(desc, p));
  DART_TRY(replan_first_read(p));
  *waves = p.ks_waves;
  *split = p.ks_split;
  return DART_OK;
}

dart_status dart_select_pivots(const dart_desc* desc, const void* X, const void* crit,
                               int32_t crit_D, int64_t crit_ld, int32_t* piv, float* l1_out,
                               void* ws, size_t ws_bytes, void* stream) {
  Plan p;
  DART_TRY(make_plan(desc, p));
  if (p.g.mode == kGiven) return DART_ERR_DTYPE;  // nothing to select
  if (p.g.B == 0) return DART_OK;
  if (!X || !piv) return DART_ERR_NULL;
  if (misaligned16(X)) return DART_ERR_ALIGN;
  if (p.g.mode == kRandom) crit = nullptr;
  DART_TRY(check_crit(p, X, crit, crit_D, crit_ld));
  DART_TRY(check_ws(p, ws, ws_bytes));
  hipStream_t st = static_cast<hipStream_t>(stream);
  float* l1 = l1_out ? l1_out : at<float>(ws, p.o_l1);
  const bool norm_pass = p.g.mode != kRandom && p.g.Pin > 0;
  if (!norm_pass) DART_TRY(launch_prepare(p, ws, st));
  if (p.g.mode == kRandom) {  // no criterion is read and l1_out is left as it is
    DART_TRY(launch_random_pivots(p, piv, st));
  } else if (norm_pass) {
    DART_TRY(launch_row_l1(p, crit, crit_D, crit_ld, l1, false, ws, st));
    DART_TRY(launch_select_pivots(p, X, crit, crit_D, crit_ld, l1, nullptr, piv, nullptr, ws, st));
  }
  if (p.g.Pe > 0 && !norm_pass) DART_TRY(launch_pivot_norms(p, X, piv, piv, ws, st));  // (their marks)
  return DART_OK;
}

dart_status dart_duplication_scores(const dart_desc* desc, const void* X, const int32_t* piv,
                                    float* S, void* ws, size_t ws_bytes, void* stream) {
  Plan p;
  DART_TRY(make_plan(desc, p));
  if (p.g.B == 0) return DART_OK;
  if (!X || !piv || !S) return DART_ERR_NULL;
  if (misaligned16(X)) return DART_ERR_ALIGN;
  DART_TRY(check_ws(p, ws, ws_bytes));
  DART_TRY(replan_first_read(p));
  hipStream_t st = static_cast<hipStream_t>(stream);
  DART_TRY(launch_prepare(p, ws, st));
  DART_TRY(launch_given_status(p, piv, ws, st));
  DART_TRY(launch_pivot_norms(p, X, piv, nullptr, ws, st));
  return launch_scores(p, X, piv, S, ws, st);
}

dart_status dart_topk_keep(const dart_desc* desc, const float* S, const int32_t* piv,
                           const void* X, int32_t* keep, int32_t* cu_keep, void* ws,
                           size_t ws_bytes, void* stream) {
  Plan p;
  DART_TRY(make_plan(desc, p));
  if (p.g.B == 0) return DART_OK;
  if (!S || !piv || !keep) return DART_ERR_NULL;
  if (X && misaligned16(X)) return DART_ERR_ALIGN;
  DART_TRY(check_ws(p, ws, ws_bytes));
  hipStream_t st = static_cast<hipStream_t>(stream);
  DART_TRY(launch_prepare(p, ws, st));
  DART_TRY(launch_given_status(p, piv, ws, st));
  DART_TRY(launch_order(p, S, ws, st));
  return launch_retain(p, S, piv, X, keep, cu_keep, ws, st, false);
}

dart_status dart_gather_compact(const dart_desc* desc, const void* X, const int64_t* pos,
                                const int32_t* keep, void* Y, int64_t* pos_out, void* ws,
                                size_t ws_bytes, void* stream) {
  Plan p;
  DART_TRY(make_plan(desc, p));
  if (p.g.B == 0) return DART_OK;
  if (!X || !keep || !Y || (pos != nullptr) != (pos_out != nullptr)) return DART_ERR_NULL;
  if (misaligned16(X) || misaligned16(Y)) return DART_ERR_ALIGN;
  DART_TRY(check_ws(p, ws, ws_bytes));
  hipStream_t st = static_cast<hipStream_t>(stream);
  DART_TRY(launch_prepare(p, ws, st));
  DART_TRY(launch_given_status(p, nullptr, ws, st));
  return launch_gather(p, X, pos, keep, Y, pos_out, st);
}

dart_status dart_compact_sequences(const dart_desc* desc, const int32_t* seq_cu,
                                   const int32_t* keep, int32_t n_tensors,
                                   const dart_row_tensor* tensors, const int64_t* pos,
                                   int32_t pos_planes, int64_t pos_plane_stride, int64_t* pos_out,
                                   int64_t pos_out_plane_stride, int32_t* seq_cu_out,
                                   int32_t* row_map, void* ws, size_t ws_bytes, void* stream) {
  Plan p;
  DART_TRY(make_plan(desc, p));
  if (!desc->span_start) return DART_ERR_NULL;  // sequences exist only around spans
  if (n_tensors < 0 || pos_planes < 0) return DART_ERR_SHAPE;
  if (!seq_cu || !keep || !seq_cu_out || !row_map || (n_tensors > 0 && !tensors) ||
      (pos_planes > 0 && (!pos || !pos_out)))
    return DART_ERR_NULL;
  for (int i = 0; i < n_tensors; ++i) {
    const dart_row_tensor& t = tensors[i];
    if (!t.src || !t.dst) return DART_ERR_NULL;
    if (t.row_bytes <= 0 || t.src_ld_bytes < t.row_bytes || t.dst_ld_bytes < t.row_bytes)
      return DART_ERR_SHAPE;
    if (misaligned16(t.src) || misaligned16(t.dst) || t.row_bytes % 16 || t.src_ld_bytes % 16 ||
        t.dst_ld_bytes % 16)
      return DART_ERR_ALIGN;
  }
  if (pos_planes > 0 && (pos_plane_stride < p.g.x_rows || pos_out_plane_stride < 0))
    return DART_ERR_SHAPE;
  DART_TRY(check_ws(p, ws, ws_bytes));
  hipStream_t st = static_cast<hipStream_t>(stream);
  DART_TRY(launch_prepare(p, ws, st, seq_cu, seq_cu_out));
  DART_TRY(launch_given_status(p, nullptr, ws, st));
  // every sequence loses its pruned vision tokens; at most this many rows remain
  const long rows_bound = (long)p.g.x_rows - p.g.total_N + p.keep_rows_bound;
  if (p.g.B == 0 || rows_bound <= 0) return DART_OK;
  SeqPos sp = {reinterpret_cast<const long long*>(pos), reinterpret_cast<long long*>(pos_out),
               (long)pos_plane_stride, (long)pos_out_plane_stride, pos_planes};
  long widest = 0;
  for (int i = 0; i < n_tensors; ++i) widest = std::max(widest, (long)tensors[i].row_bytes);
  const bool mapped = n_tensors == 0 || (p.g.B > kSeqMapped && widest > 1024);
  if (mapped) {
    DART_LAUNCH(k_seq_row_map, dim3((unsigned)((rows_bound + 255) / 256)), dim3(256), 0, st, p.g,
                seq_cu, seq_cu_out, keep, row_map, sp);
    DART_LAUNCH_CHECK();
  }
  for (int i0 = 0; i0 < n_tensors; i0 += kSeqOps) {
    SeqOps ops = {};
    const int cnt = std::min(n_tensors - i0, kSeqOps);
    long longest = 0;
    for (int i = 0; i < cnt; ++i) {
      const dart_row_tensor& t = tensors[i0 + i];
      ops.src[i] = static_cast<const unsigned char*>(t.src);
      ops.dst[i] = static_cast<unsigned char*>(t.dst);
      ops.row_bytes[i] = t.row_bytes;
      ops.src_ld[i] = t.src_ld_bytes;
      ops.dst_ld[i] = t.dst_ld_bytes;
      longest = std::max(longest, (long)t.row_bytes);
    }
    // rows per wave (measured: see the kernel)
    const int R = mapped ? 1 : longest <= 1024 ? 4 : longest <= 2048 ? 2 : 1;
    const dim3 grid((unsigned)round_up8((rows_bound + 4 * R - 1) / (4 * R)), cnt);
#define DART_LAUNCH_SEQ(ROWS, MAPPED)                                                            \
  DART_LAUNCH((k_gather_rows<ROWS, MAPPED>), grid, dim3(256), 0, st, p.g, ops, i0 == 0, seq_cu,  \
              seq_cu_out, keep, row_map, sp)
    if (mapped) DART_LAUNCH_SEQ(1, true);
    else if (R == 4) DART_LAUNCH_SEQ(4, false);
    else if (R == 2) DART_LAUNCH_SEQ(2, false);
    else DART_LAUNCH_SEQ(1, false);
#undef DART_LAUNCH_SEQ
    DART_LAUNCH_CHECK();
  }
  return DART_OK;
}

dart_status dart_reduce(const dart_desc* desc, const void* X, const void* crit, int32_t crit_D,
                        int64_t crit_ld, const int64_t* pos, void* Y, int64_t* pos_out,
                        int32_t* keep, int32_t* cu_keep, int32_t* piv_out, float* S_out, void* ws,
                        size_t ws_bytes, void* stream) {
  return reduce_impl(desc, X, crit, crit_D, crit_ld, pos, Y, pos_out, keep, cu_keep, piv_out,
                     S_out, ws, ws_bytes, stream, nullptr);
}

dart_status dart_reduce_profiled(const dart_desc* desc, const void* X, const void* crit,
                                 int32_t crit_D, int64_t crit_ld, const int64_t* pos, void* Y,
                                 int64_t* pos_out, int32_t* keep, int32_t* cu_keep,
                                 int32_t* piv_out, float* S_out, void* ws, size_t ws_bytes,
                                 void* stream, void* const* events) {
  if (!events) return DART_ERR_NULL;
  for (int k = 0; k < 12; ++k)
    if (!events[k]) return DART_ERR_NULL;
  return reduce_impl(desc, X, crit, crit_D, crit_ld, pos, Y, pos_out, keep, cu_keep, piv_out,
                     S_out, ws, ws_bytes, stream, events);
}

dart_status dart_reduce_with_norms(const dart_desc* desc, const void* X, const void* crit,
                                   int32_t crit_D, int64_t crit_ld, const float* l1,
                                   double l1_rel_err, const int64_t* pos, void* Y,
                                   int64_t* pos_out, int32_t* keep, int32_t* cu_keep,
                                   int32_t* piv_out, float* S_out, void* ws, size_t ws_bytes,
                                   void* stream) {
  if (!l1) return DART_ERR_NULL;
  return reduce_impl(desc, X, crit, crit_D, crit_ld, pos, Y, pos_out, keep, cu_keep, piv_out,
                     S_out, ws, ws_bytes, stream, nullptr, l1, l1_rel_err);
}

size_t dart_static_scratch_bytes(void) { return kStaticScratchBytes; }

dart_status dart_reduce_static(const dart_desc* desc, const void* X, const void* crit,
                               int32_t crit_D, int64_t crit_ld, const int64_t* pos, void* Y,
                               int64_t* pos_out, int32_t* keep, int32_t* cu_keep,
                               int32_t* piv_out, float* S_out, void* stream) {
  Plan p;
  DART_TRY(make_plan(desc, p));
  if (p.total > kStaticScratchBytes) return DART_ERR_STATIC_LIMIT;
  void* ws = nullptr;
  DART_TRY(static_scratch(&ws));
  return reduce_impl(desc, X, crit, crit_D, crit_ld, pos, Y, pos_out, keep, cu_keep, piv_out,
                     S_out, ws, kStaticScratchBytes, stream, nullptr);
}

dart_status dart_device_status_static(const dart_desc* desc, void* stream) {
  void* ws = nullptr;
  DART_TRY(static_scratch(&ws));
  return dart_device_status(desc, ws, stream);
}

dart_status dart_device_status(const dart_desc* desc, const void* ws, void* stream) {
  Plan p;
  DART_TRY(make_plan(desc, p));
  if (!ws) return DART_ERR_WORKSPACE;
  if (p.g.B == 0 || (p.g.cu == nullptr && p.g.mode != kGiven && !p.fusable)) return DART_OK;
  // [0] ragged offsets / budgets / spans, [1] given pivots, [2] sequences around the spans,
  // [3] the one-launch path gave up a bounded wait (its outputs are then unspecified)
  int flag[4] = {0, 0, 0, 0};
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (hipMemcpyAsync(flag, static_cast<const unsigned char*>(ws) + p.o_status, sizeof(flag),
                     hipMemcpyDeviceToHost, st) != hipSuccess)
    return DART_ERR_HIP;
  if (hipStreamSynchronize(st) != hipSuccess) return DART_ERR_HIP;
  if (p.g.cu == nullptr) flag[0] = 0;
  if (p.g.mode != kGiven) flag[1] = 0;
  if (p.g.span == nullptr) flag[2] = 0;
  flag[3] = (p.fusable && flag[3] == kFuAborted) ? 1 : 0;
  return (flag[0] | flag[1] | flag[2] | flag[3]) ? DART_ERR_DEVICE : DART_OK;
}

dart_status dart_probe_mfma_dot32(const void* A, const void* B, float* out, int32_t tiles,
                                  void* stream) {
  if (tiles < 0) return DART_ERR_SHAPE;
  if (tiles == 0) return DART_OK;
  if (!A || !B || !out) return DART_ERR_NULL;
  if (misaligned16(A) || misaligned16(B) || misaligned16(out)) return DART_ERR_ALIGN;
  DART_LAUNCH(k_probe_mfma_dot32, dim3(tiles), dim3(64), 0, static_cast<hipStream_t>(stream),
              static_cast<const unsigned char*>(A), static_cast<const unsigned char*>(B),
              out);
  DART_LAUNCH_CHECK();
  return DART_OK;
}

double dart_score_tolerance(int32_t dtype) {
  return score_abs_bound(dtype == DART_BF16 ? kBF16 : kF32);
}

const char* dart_strerror(dart_status status) {
  switch (status) {
    case DART_OK: return "ok";
    case DART_ERR_NULL: return "a required pointer is NULL";
    case DART_ERR_SHAPE: return "a size or stride is out of range";
    case DART_ERR_BUDGET: return "the keep budget violates P <= K <= N";
    case DART_ERR_DTYPE: return "unknown dtype or pivot mode";
    case DART_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case DART_ERR_ALIGN: return "row starts are not 16-byte aligned";
    case DART_ERR_HIP: return "a HIP call or kernel launch failed";
    case DART_ERR_STATIC_LIMIT:
      return "the problem needs more scratch than the built-in buffer of dart_reduce_static "
             "holds (dart_static_scratch_bytes); use dart_reduce with a workspace";
    case DART_ERR_DEVICE:
      return "a ragged sample violated the size or budget limits, a span or sequence is invalid, "
             "or a given pivot list is invalid";
  }
  return "unknown status";
}

}  // extern "C"
