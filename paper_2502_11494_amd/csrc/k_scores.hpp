// Duplication scores of Definition 2 / Eq. (7): the cosine between every pivot
// and every token of its sample.
//
// bf16 hidden states: the tokens x pivots x D contraction runs on the matrix
// cores (v_mfma_f32_16x16x32_bf16).  A workgroup of W waves in KS groups owns
// 16*W/KS token rows; a wave owns 16 of them and walks its group's share of D in
// chunks of 128 elements:
//   HBM -> registers (four rows per load instruction, 256 B contiguous each, one
//       chunk ahead) -> LDS (row-padded) -> MFMA A fragments (ds_read_b128,
//       conflict-free).
// The pivot rows of the chunk are staged once per group in LDS (double buffered)
// and serve as B fragments.  The squared token norms come from the norm pass
// when it has read the same rows; otherwise the token fragment is fed as both
// operands, which yields the tile's Gram matrix, whose diagonal is |x_j|^2, at
// no extra memory traffic.  Every MFMA starts from a zero accumulator and its
// 32-term sums are added up in fp64 on the vector ALU.  bf16 x bf16 products are
// exact in fp32, so the only rounding is inside the matrix core's 32-term sum:
// see score_abs_bound().
//
// fp32 hidden states: the same contraction on the fp64 matrix instructions (products of two
// floats are exact in fp64): see "fp32 score tiles" below.
#pragma once
#include "common.hpp"

namespace dart {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Absolute bound on |stored fp32 score - exact cosine|.
// bf16: one MFMA returns the sum of 32 exact products with an error of at most
// kMfmaUlps * 2^-24 times the sum of their magnitudes.  The matrix core's internal
// rounding is not documented; measured over millions of random, wide-range and
// cancelling inputs the worst case is 6 * 2^-24, and 16 is assumed here.  The
// partial sums are added in fp64, so the dot product errs by at most
// 16 * 2^-24 * sum|p_d x_d| <= 16 * 2^-24 |p||x|.  The token norm comes from the
// same kind of sum and enters through a square root (half the relative error).
// Two more units for rounding the quotient to fp32 and the fp64 steps.
// fp32 inputs: all fp64, only the final rounding to fp32 counts.
// The token norms may also come from elsewhere: from the norm pass, in fp64, or from the one-launch
// kernel's fp32 squares (relative error 3.5 * 2^-24 on the square, half of it on the norm; 2 units).
constexpr double kMfmaUlps = 16.0;
enum TokenNorms { kNormsGram, kNormsF64, kNormsF32Squares };
inline double score_abs_bound(int dtype, TokenNorms norms = kNormsGram) {
  const double u = 5.9604644775390625e-08;  // 2^-24
  if (dtype != kBF16) return 4.0 * u;
  return (norms == kNormsGram ? kMfmaUlps * 1.5 + 2.0
                              : kMfmaUlps + 2.0 + (norms == kNormsF64 ? 0.0 : 2.0)) * u;
}

// Tile -> (sample, tile inside the sample).  Returns false for surplus blocks.
__device__ __forceinline__ bool locate_tile(const Geo& g, int tile, int& b, int& tl) {
  if (g.cu == nullptr) {
    int tps = (g.N + g.tile_rows - 1) / g.tile_rows;
    b = tile / tps;
    tl = tile - b * tps;
    return b < g.B;
  }
  if (tile >= g.tile_start[g.B]) return false;
  b = last_at_most(g.tile_start, g.B, tile);
  tl = tile - g.tile_start[b];
  return true;
}

// Scores of one wave's 16 rows from the accumulated dot products and Gram diagonal.
// Output tile: lane holds column (lane&15) and rows 4*(lane>>4)..+3 of each 16x16 block.
// With tokens as the A operand, rows are tokens and columns are pivots (Gram: columns are
// tokens too, so |x_m|^2 sits in lane (m/4)*16+m, slot m%4).
// xnorm (the wave's 16 rows; nullptr: from the Gram diagonal) and pnorm [NB*16]: norms, in LDS.
// put(nb, s): receives the lane's four scores against pivot 16 nb + (lane & 15).
template <int NB, typename Put>
__device__ __forceinline__ void finish_scores(int lane, const double (&acc64)[NB][4],
                                              const double (&gram64)[4], const double* xnorm,
                                              const double* pnorm, const Put& put) {
  const int g4 = lane >> 4;
  double xn[4];
#pragma unroll
  for (int r = 0; r < 4; ++r)
    xn[r] = xnorm ? xnorm[g4 * 4 + r] : sqrt(__shfl(gram64[r], g4 * 16 + g4 * 4 + r, kWave));
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const double pn = pnorm[nb * 16 + (lane & 15)];
    f32x4v s;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double den = pn * xn[r];
      s[r] = (float)(den > 0.0 ? acc64[nb][r] / den : 0.0) + 0.0f;
    }
    put(nb, s);
  }
}

// ---- bf16 score tiles ------------------------------------------------------------------------
// The WAVES waves of a workgroup form KS groups that share the same 16*WAVES/KS token rows;
// group gk walks the D-chunks [gk*chunks/KS, (gk+1)*chunks/KS) with its own pivot chunks, and
// the groups' partial sums are added in group order at the end.  A tile of few rows (many tiles:
// every compute unit busy, a sample's scores done early) then still has WAVES waves' worth of
// loads in flight, at the pivot traffic of its row count.  KS = 1 is the plain tile of 16*WAVES
// rows.
constexpr int kKsCH = 128;  // elements of D per chunk

// LDS: token chunks of the waves, pivot chunks of the KS groups (double buffered), the norms of
// the tile's rows and of the pivots.  Rows are padded by 16 bytes so that the 16-row x 64-byte fragment
// reads hit distinct banks.  After the last chunk the groups' partial sums (kPartB bytes per
// wave of the groups 1..KS-1) overlay a and, for the widest shapes, the start of p.
template <int NB, int KS, int WAVES>
struct KSplitShared {
  static constexpr int kRowB = kKsCH * 2 + 16;
  static constexpr int kPartB = kWave * (NB * 4 + 4) * 8;
  unsigned char a[WAVES * 16 * kRowB];
  unsigned char p[KS * 2 * NB * 16 * kRowB];
  double pnorm[NB * 16], xnorm[16 * WAVES / KS];
  static_assert((WAVES - WAVES / KS) * kPartB <= WAVES * 16 * kRowB + KS * 2 * NB * 16 * kRowB,
                "the groups' partial sums must fit in the token and pivot chunks they overlay");
};

// LDS bytes of a shape (host side: which shapes fit a compute unit).
constexpr size_t ksplit_lds_bytes(int NB, int KS, int WAVES) {
  return (size_t)(WAVES * 16 + KS * 2 * NB * 16) * (kKsCH * 2 + 16) +
         (size_t)(NB * 16 + 16 * WAVES / KS) * 8;
}

// Tile tl (16*WAVES/KS rows) of sample b.
// TAIL: D is not a multiple of the chunk (the last chunk's missing pieces are zeroed).
// XN: the squared token norms are given (l2sq, from the norm pass): the Gram products and
// their accumulation are left out.
// COH: piv, pl2 and l2sq were written, and S will be read, by other workgroups of this launch.
template <int NB, int KS, int WAVES, bool TAIL, bool XN, bool COH>
__device__ __forceinline__ void score_tile_ksplit(const Geo& g, const Sample& sm, int b, int tl,
                                                  const void* X, const int* piv, const double* pl2,
                                                  const double* l2sq, float* S,
                                                  KSplitShared<NB, KS, WAVES>& sh) {
  constexpr int ROWS = 16 * WAVES / KS;
  constexpr int WG = WAVES / KS;        // waves per group
  constexpr int TG = WG * kWave;        // threads per group
  constexpr int kRowB = kKsCH * 2 + 16;
  constexpr int PC = kKsCH / 8;         // 16-byte pieces per row per chunk
  constexpr int RPI = kWave / PC;       // rows covered by one load instruction
  constexpr int LA = 16 / RPI;          // token loads per lane per chunk
  constexpr int PP = NB * 16 * PC;      // pivot pieces per chunk
  constexpr int LP = (PP + TG - 1) / TG;
  constexpr int KSTEPS = kKsCH / 32;    // matrix-core steps per chunk
  constexpr int PV = NB * 4 + (XN ? 0 : 4);  // partial sums per lane
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int gk = wave / WG, wi = wave - gk * WG, tg = tid - gk * TG;
  const int n = sm.n, P = g.P;
  // What the tile waits for is requested in the order of its need: the pivots' indices, the
  // norms, the first rows, and, once the indices are there, the first pivot pieces.
  // pivot pieces: piece id = tg + TG*k -> pivot row id/PC, piece id%PC (== lane%PC); padding
  // slots read the sample's first row and are zeroed when the registers go to LDS
  int pidx[LP];
#pragma unroll
  for (int k = 0; k < LP; ++k) {
    const int i = (tg + TG * k) / PC;
    pidx[k] = i < g.Pin ? ld_dev<COH>(&piv[b * P + i]) : 0;
  }
  constexpr int XR = XN ? ROWS : 0;  // the norms: a thread each, the rows' first
  static_assert(ROWS + NB * 16 <= WAVES * kWave, "a norm per thread");
  double l2 = 0.0;
  if (tid < XR) {
    const int j = tl * ROWS + tid;
    l2 = ld_dev<COH>(&l2sq[sm.row0 + (j < n ? j : n - 1)]);
  } else if (tid < XR + NB * 16) {
    l2 = ld_dev<COH>(&pl2[b * g.Ppad + (tid - XR)]);
  }

  const long rowbytes = g.ld * 2;
  const unsigned char* Xb = static_cast<const unsigned char*>(X) + (long)sm.xrow * rowbytes;
  const int pieces = g.D / 8;
  const int chunks_all = (g.D + kKsCH - 1) / kKsCH;
  const int c_first = gk * chunks_all / KS, c_end = (gk + 1) * chunks_all / KS;
  const int my_cnt = c_end - c_first;
  const int max_cnt = (chunks_all + KS - 1) / KS;  // every group runs this many rounds
  const int col16 = lane % PC, rowsub = lane / PC;
  const int j0 = tl * ROWS + wi * 16;
  const u32x4 zero = {0u, 0u, 0u, 0u};

  const unsigned char* aptr[LA];
#pragma unroll
  for (int t = 0; t < LA; ++t) {
    int r = j0 + t * RPI + rowsub;
    r = r < n ? r : n - 1;  // rows past the sample's end re-read its last row; never stored
    aptr[t] = Xb + (long)r * rowbytes + (TAIL ? 0 : col16 * 16);
  }
  // With TAIL the lane's column offset is added per chunk instead: a piece past the end of
  // the row must re-read the row's first 16 bytes, not bytes behind a row shorter than a chunk
  const int tail_col = TAIL ? col16 * 16 : 0;
  u32x4 ra[LA], rp[LP];
  auto chunk_offset = [&](int c) -> long {
    const bool in = !TAIL || c * PC + col16 < pieces;
    return in ? (long)c * (kKsCH * 2) + tail_col : 0;
  };
  auto load_rows = [&](long off) {
#pragma unroll
    for (int t = 0; t < LA; ++t)
      ra[t] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(aptr[t] + off));
  };
  const int c0 = my_cnt > 0 ? c_first : 0;
  load_rows(chunk_offset(c0));
  // (global pointers by type: through a generic one the loads are flat ones, which also count as
  // LDS operations, so that the barrier and the LDS store of a chunk wait for every load in
  // flight: 16 images of 576 tokens in tiles of 96 rows 23.4 us, 21.7 this way)
  typedef const __attribute__((address_space(1))) unsigned char global_bytes;
  typedef const __attribute__((address_space(1))) u32x4 global_piece;
  global_bytes* pptr[LP];
  bool preal[LP], pmine[LP];
#pragma unroll
  for (int k = 0; k < LP; ++k) {
    const int pid = tg + TG * k, i = pid / PC;
    pmine[k] = pid < PP;
    preal[k] = i < P;
    const unsigned char* pr = Xb;
    if (i < g.Pin) {
      const int q = pidx[k] < 0 ? 0 : (pidx[k] < n ? pidx[k] : n - 1);
      pr = Xb + (long)q * rowbytes;
    } else if (i < P) {
      pr = static_cast<const unsigned char*>(g.E) + ((long)b * g.Pe + (i - g.Pin)) * g.lde * 2;
    }
    pptr[k] = (global_bytes*)(pr + (TAIL ? 0 : col16 * 16));
  }
  auto load_pivots = [&](long off) {
#pragma unroll
    for (int k = 0; k < LP; ++k) rp[k] = *(global_piece*)(pptr[k] + off);
  };
  load_pivots(chunk_offset(c0));
  if (tid < XR) sh.xnorm[tid] = sqrt(l2);
  else if (tid < XR + NB * 16) sh.pnorm[tid - XR] = sqrt(l2);
  unsigned char* la = sh.a + wave * (16 * kRowB);
  unsigned char* lpg = sh.p + gk * (2 * NB * 16 * kRowB);
  const int frag_off = (lane & 15) * kRowB + (lane >> 4) * 16;
  const f32x4 fzero = {0.f, 0.f, 0.f, 0.f};

  double acc64[NB][4], gram64[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    gram64[r] = 0.0;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc64[nb][r] = 0.0;
  }

  // chunk c of this group (clamped to a chunk it owns, so that every load is unconditional
  // and in bounds; the surplus rounds of a group with fewer chunks compute nothing).  The
  // chunk's pivot pieces are requested just before its token pieces (vector loads return in
  // order), and nothing touches a load's result while it is in flight.
  auto load_chunk = [&](int c) {
    load_pivots(chunk_offset(c));
    load_rows(chunk_offset(c));
  };
  auto store_p = [&](int c, int buf) {
    const bool in = !TAIL || c * PC + col16 < pieces;
#pragma unroll
    for (int k = 0; k < LP; ++k)
      if (pmine[k])
        *reinterpret_cast<u32x4*>(lpg + buf * (NB * 16 * kRowB) + ((tg + TG * k) / PC) * kRowB +
                                  col16 * 16) = (in && preal[k]) ? rp[k] : zero;
  };
  const int c_last = my_cnt > 0 ? c_end - 1 : 0;
  store_p(c_first, 0);
  for (int it = 0; it < max_cnt; ++it) {
    const int c = c_first + it;
    const bool live = it < my_cnt;
    {
      // the wave's rows go registers -> its own LDS region (LDS operations of one wave
      // complete in order, so the fragment reads below need no barrier of their own)
      const bool in = !TAIL || c * PC + col16 < pieces;
#pragma unroll
      for (int t = 0; t < LA; ++t)
        *reinterpret_cast<u32x4*>(la + (t * RPI + rowsub) * kRowB + col16 * 16) =
            (in && live) ? ra[t] : zero;
    }
    const bool more = it + 1 < my_cnt;
    if (it + 1 < max_cnt) load_chunk(more ? c + 1 : c_last);
    __syncthreads();  // pivot buffer it%2 is complete; buffer (it+1)%2 is no longer read
    const unsigned char* lp = lpg + (it & 1) * (NB * 16 * kRowB);
    if (live) {
#pragma unroll
      for (int s = 0; s < KSTEPS; ++s) {
        const bf16x8 af = *reinterpret_cast<const bf16x8*>(la + frag_off + s * 64);
        f32x4 gram = fzero;
        if (!XN) gram = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, af, fzero, 0, 0, 0);
        f32x4 acc[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          const bf16x8 pf =
              *reinterpret_cast<const bf16x8*>(lp + nb * (16 * kRowB) + frag_off + s * 64);
          acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, pf, fzero, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (!XN) gram64[r] += (double)gram[r];
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) acc64[nb][r] += (double)acc[nb][r];
        }
      }
    }
    if (it + 1 < max_cnt) store_p(more ? c + 1 : c_last, (it + 1) & 1);
  }
  if (KS > 1) {
    // the groups' partial sums: groups 1.. leave theirs in LDS (over the chunks, which nobody
    // reads any more), group 0 adds them in group order
    __syncthreads();
    double* part = reinterpret_cast<double*>(sh.a);
    if (gk > 0) {
      double* out = part + ((long)((gk - 1) * WG + wi) * kWave + lane) * PV;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int r = 0; r < 4; ++r) out[nb * 4 + r] = acc64[nb][r];
      if (!XN) {
#pragma unroll
        for (int r = 0; r < 4; ++r) out[NB * 4 + r] = gram64[r];
      }
    }
    __syncthreads();
    if (gk == 0) {
#pragma unroll
      for (int o = 1; o < KS; ++o) {
        const double* in = part + ((long)((o - 1) * WG + wi) * kWave + lane) * PV;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc64[nb][r] += in[nb * 4 + r];
        if (!XN) {
#pragma unroll
          for (int r = 0; r < 4; ++r) gram64[r] += in[NB * 4 + r];
        }
      }
    }
  }
  if (gk != 0 || j0 >= n) return;
  const double* xn = XN ? sh.xnorm + wi * 16 : nullptr;
  const int r0 = (lane >> 4) * 4;
  float* Sb = S + (long)P * sm.row0;
  const int j = j0 + r0;
  // four neighbouring scores in one store where that is aligned
  const bool by4 = !COH && (n & 3) == 0 && (reinterpret_cast<uintptr_t>(Sb) & 15u) == 0;
  finish_scores<NB>(lane, acc64, gram64, xn, sh.pnorm, [&](int nb, const f32x4v& s) {
    const int i = nb * 16 + (lane & 15);
    float* out = Sb + (long)i * n + j;
    if (i >= P || j >= n) return;
    if (by4) {
      *reinterpret_cast<f32x4v*>(out) = s;
      return;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (j + r < n) st_dev<COH>(out + r, s[r]);
  });
}

// grid: the tiles of g.tile_rows = 16*WAVES/KS rows (dense: B*ceil(N/rows); ragged: an upper
// bound), rounded up to a multiple of 8 blocks (a die per contiguous eighth of the tiles);
// WAVES*64 threads.  NB = Ppad/16 pivot column blocks.
template <int NB, int KS, int WAVES, bool TAIL, bool XN>
__global__ __launch_bounds__(WAVES * 64) void k_scores_ksplit(Geo g, const void* __restrict__ X,
                                                       const int* __restrict__ piv,
                                                       const double* __restrict__ pl2,
                                                       const double* __restrict__ l2sq,
                                                       float* __restrict__ S) {
  __shared__ __align__(16) KSplitShared<NB, KS, WAVES> sh;
  int b, tl;
  const int tile = (int)xcd_contiguous(blockIdx.x, gridDim.x);
  if (!locate_tile(g, tile, b, tl)) return;
  const Sample sm = sample_of(g, b);
  if (sm.k == 0 || tl * (16 * WAVES / KS) >= sm.n) return;
  score_tile_ksplit<NB, KS, WAVES, TAIL, XN, false>(g, sm, b, tl, X, piv, pl2, l2sq, S, sh);
}

// ---- fp32 score tiles ------------------------------------------------------------------------
// fp32 hidden states: the contraction runs on the fp64 matrix instructions (the product of two
// floats is exact in fp64, the sums are fp64 throughout).  A lane loads four consecutive elements
// of its row; element e of every lane feeds the e-th of four matrix instructions (the order of D
// inside an instruction is free as long as both operands agree).  The waves of a workgroup split D
// and their partial sums are added in wave order, so a score is a function of the two rows' bytes.
//
// Many rows (k_scores_f32_t16): blocks of 16 rows by 16 pivots, v_mfma_f64_16x16x4 (64 cycles);
// X is read once and a pivot piece serves all rows of the tile.  A compute unit takes in about
// 35-50 GB/s from memory and the pivots' pieces queue with the rows' (every workgroup reads all of
// them once), so the kernel runs at the speed of the unit with the most rows plus pivots: tiles of
// up to 32 rows, the height chosen on the host so that the units share the rows evenly
// (f32_tile_rows).  5780 rows of 2048 by 16 pivots: 74 us -> 20 us (47 MB of rows); the vector-ALU
// kernel this replaces held 4 rows by 8 pivots per workgroup, read X once per 8 pivots and every
// pivot once per 4 rows.
constexpr int kF32Waves = 8;
typedef double f64x4 __attribute__((ext_vector_type(4)));

template <int NB, int RB>
struct F32TileShared {
  double part[kF32Waves][RB][NB][4][kWave];
  double xx[kF32Waves][RB][kWave];
};

// grid: tiles of g.tile_rows <= 16*RB rows; 512 threads.  Result layout of the instruction: lane l,
// slot r holds row (l >> 4) + 4 r, column l & 15.
template <int NB, int RB>
__global__ __launch_bounds__(kF32Waves * 64) void k_scores_f32_t16(
    Geo g, const void* __restrict__ X, const int* __restrict__ piv,
    const double* __restrict__ pl2, float* __restrict__ S) {
  constexpr int kRing = NB * RB <= 2 ? 2 : 1;  // steps in flight
  __shared__ F32TileShared<NB, RB> sh;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int b, tl;
  if (!locate_tile(g, blockIdx.x, b, tl)) return;
  const Sample sm = sample_of(g, b);
  const int n = sm.n, P = g.P, j0 = tl * g.tile_rows;
  if (sm.k == 0 || j0 >= n) return;
  const int rows = n - j0 < g.tile_rows ? n - j0 : g.tile_rows;
  const int r16 = lane & 15, g4 = lane >> 4;
  // A step is a 128-byte line of every row, two 16-byte pieces per lane.
  const int pieces = g.D / 4;                // 16-byte pieces per row
  const int steps = pieces / 8;              // whole steps
  const int s0 = wave * steps / kF32Waves, cnt = (wave + 1) * steps / kF32Waves - s0;
  const f32x4v* xr[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    int r = rb * 16 + r16;
    r = j0 + (r < rows ? r : rows - 1);  // rows past the end re-read the last; never stored
    xr[rb] = reinterpret_cast<const f32x4v*>(static_cast<const float*>(X) + ((long)sm.xrow + r) * g.ld);
  }
  const f32x4v* pr[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int i = nb * 16 + r16 < P ? nb * 16 + r16 : P - 1;  // columns past P: never stored
    pr[nb] = reinterpret_cast<const f32x4v*>(pivot_row(g, X, 4, sm, b, i, piv));
  }
  f32x4v ra[kRing][RB][2], rp[kRing][NB][2];
  auto load = [&](int slot, int s) {  // step s of this wave's share
    const int t = (s0 + s) * 8 + g4;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int h = 0; h < 2; ++h) ra[slot][rb][h] = xr[rb][t + h * 4];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int h = 0; h < 2; ++h) rp[slot][nb][h] = pr[nb][t + h * 4];
  };
  // two chains per sum: a matrix instruction that adds to the previous one's result waits for it
  f64x4 acc[RB][NB], acc_odd[RB][NB];
  double xx[RB], xx_odd[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    xx[rb] = xx_odd[rb] = 0.0;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[rb][nb] = acc_odd[rb][nb] = f64x4{0.0, 0.0, 0.0, 0.0};
  }
  auto use = [&](const f32x4v (&x)[RB][2], const f32x4v (&p)[NB][2]) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int e = 0; e < 4; e += 2) {
        double p0[NB], p1[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          p0[nb] = (double)p[nb][h][e];
          p1[nb] = (double)p[nb][h][e + 1];
        }
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          const double a0 = (double)x[rb][h][e], a1 = (double)x[rb][h][e + 1];
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) {
            acc[rb][nb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, p0[nb], acc[rb][nb], 0, 0, 0);
            acc_odd[rb][nb] =
                __builtin_amdgcn_mfma_f64_16x16x4f64(a1, p1[nb], acc_odd[rb][nb], 0, 0, 0);
          }
          xx[rb] = fma(a0, a0, xx[rb]);
          xx_odd[rb] = fma(a1, a1, xx_odd[rb]);
        }
      }
  };
#pragma unroll
  for (int u = 0; u < kRing; ++u)
    if (u < cnt) load(u, u);
  int s = 0;
  for (; s + 2 * kRing <= cnt; s += kRing) {
#pragma unroll
    for (int u = 0; u < kRing; ++u) {
      use(ra[u], rp[u]);
      load(u, s + kRing + u);
    }
  }
#pragma unroll
  for (int u = 0; u < kRing; ++u)
    if (s + u < cnt) {
      use(ra[u], rp[u]);
      if (s + kRing + u < cnt) load(u, s + kRing + u);
    }
#pragma unroll
  for (int u = 0; u < kRing - 1; ++u)
    if (s + kRing + u < cnt) use(ra[u], rp[u]);
  // the incomplete step of a row whose pieces are no multiple of eight belongs to the last wave
  // (missing pieces: both operands zero, so that nothing meets what piece 0 holds)
  if (wave == kF32Waves - 1 && steps * 8 < pieces) {
    const f32x4v fz = {0.f, 0.f, 0.f, 0.f};
    f32x4v x[RB][2], p[NB][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int t = steps * 8 + h * 4 + g4;
      const bool in = t < pieces;
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        x[rb][h] = xr[rb][in ? t : 0];
        x[rb][h] = in ? x[rb][h] : fz;
      }
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        p[nb][h] = pr[nb][in ? t : 0];
        p[nb][h] = in ? p[nb][h] : fz;
      }
    }
    use(x, p);
  }
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int r = 0; r < 4; ++r) sh.part[wave][rb][nb][r][lane] = acc[rb][nb][r] + acc_odd[rb][nb][r];
    sh.xx[wave][rb][lane] = xx[rb] + xx_odd[rb];
  }
  __syncthreads();
  float* Sb = S + (long)P * sm.row0;
  for (int o = tid; o < RB * NB * 256; o += kF32Waves * 64) {
    const int m = o & 15, rb = (o >> 4) % RB, i = o / (16 * RB);  // token row, pivot
    const int src = (m & 3) * 16 + (i & 15);
    double d = 0.0, x2 = 0.0;
#pragma unroll
    for (int w = 0; w < kF32Waves; ++w) {
      d += sh.part[w][rb][i >> 4][m >> 2][src];
      const double* q = sh.xx[w][rb];
      x2 += (q[m] + q[16 + m]) + (q[32 + m] + q[48 + m]);
    }
    if (i < P && rb * 16 + m < rows) {
      const double den = sqrt(pl2[b * g.Ppad + i]) * sqrt(x2);
      Sb[(long)i * n + j0 + rb * 16 + m] = (float)(den > 0.0 ? d / den : 0.0) + 0.0f;
    }
  }
}

// Few rows (k_scores_f32_t4): tiles of 4 rows by 4 PG pivots, so that one 576-token image gives
// hundreds of workgroups; v_mfma_f64_4x4x4 (four independent 4x4x4 blocks, 16 cycles).  Of the blocks
// PG are groups of four pivots, times 4 / PG parts of a step's pieces: with PG = 1 a workgroup takes in
// the fewest pivot rows and a load's neighbouring lanes are neighbours in memory, with PG = 4 the
// fewest workgroups read a token row (f32_tile chooses).  Latency-bound (a chain of launch, pivot
// indices, rows, sums): eight steps in flight per wave.  Scores of 300 rows of 4096, stage entry point,
// with 8, 24, 64 pivots: 11.6, 16.9, 37 us; on the vector ALU 12.3, 26.9, 64 us, and 14.5, 37, 78 us
// with a workgroup per 4 rows going through all pivots.
// Operand layout: lane l holds row l & 3 of block (l >> 2) & 3, k = l >> 4; result: lane l holds
// column l & 3 of block (l >> 2) & 3, row l >> 4.
struct F32SmallShared {
  double part[kF32Waves][kWave];
  double xx[kF32Waves][kWave];
};

// grid: (tiles of 4 rows, groups of 4 PG pivots); 512 threads.
template <int PG>
__global__ __launch_bounds__(kF32Waves * 64) void k_scores_f32_t4(
    Geo g, const void* __restrict__ X, const int* __restrict__ piv,
    const double* __restrict__ pl2, float* __restrict__ S) {
  constexpr int kRing = 8, kHalves = 4 / PG, kStep = 4 * kHalves;  // pieces per step and row
  __shared__ F32SmallShared sh;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int b, tl;
  if (!locate_tile(g, blockIdx.x, b, tl)) return;
  const Sample sm = sample_of(g, b);
  if (sm.k == 0 || tl * 4 >= sm.n) return;
  const int n = sm.n, P = g.P, j0 = tl * 4;
  const int r4 = lane & 3, blk = (lane >> 2) & 3, pg = blk % PG;
  const int col = (lane >> 4) * kHalves + blk / PG;  // the lane's piece inside a step
  const int pieces = g.D / 4;
  const int steps = pieces / kStep;  // whole steps
  const int s0 = wave * steps / kF32Waves, cnt = (wave + 1) * steps / kF32Waves - s0;
  const int jr = j0 + r4 < n ? j0 + r4 : n - 1;  // rows past the end re-read the last; never stored
  const f32x4v* xr = reinterpret_cast<const f32x4v*>(static_cast<const float*>(X) +
                                                     ((long)sm.xrow + jr) * g.ld);
  const f32x4v* xs = xr + s0 * kStep + col;
  // (the incomplete step at a row's end, as above)
  const bool rest = wave == kF32Waves - 1 && steps * kStep < pieces;
  const bool rest_in = steps * kStep + col < pieces;
  const int t_rest = rest_in ? steps * kStep + col : 0;
  float* Sb = S + (long)P * sm.row0;
  const int i0 = blockIdx.y * 4 * PG;
  const int i = i0 + pg * 4 + r4 < P ? i0 + pg * 4 + r4 : P - 1;  // columns past P: never stored
  const f32x4v* pr = reinterpret_cast<const f32x4v*>(pivot_row(g, X, 4, sm, b, i, piv));
  const f32x4v* ps = pr + s0 * kStep + col;
  f32x4v ra[kRing], rp[kRing];
  auto load = [&](int slot, int s) {
    ra[slot] = xs[s * kStep];
    rp[slot] = ps[s * kStep];
  };
  double acc4[4] = {0.0, 0.0, 0.0, 0.0}, xx4[4] = {0.0, 0.0, 0.0, 0.0};  // independent chains
  auto use = [&](const f32x4v& x, const f32x4v& p) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double a = (double)x[e];
      acc4[e] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, (double)p[e], acc4[e], 0, 0, 0);
      xx4[e] = fma(a, a, xx4[e]);
    }
  };
#pragma unroll
  for (int u = 0; u < kRing; ++u)
    if (u < cnt) load(u, u);
  int s = 0;
  for (; s + 2 * kRing <= cnt; s += kRing) {
#pragma unroll
    for (int u = 0; u < kRing; ++u) {
      use(ra[u], rp[u]);
      load(u, s + kRing + u);
    }
  }
#pragma unroll
  for (int u = 0; u < kRing; ++u)
    if (s + u < cnt) {
      use(ra[u], rp[u]);
      if (s + kRing + u < cnt) load(u, s + kRing + u);
    }
#pragma unroll
  for (int u = 0; u < kRing - 1; ++u)
    if (s + kRing + u < cnt) use(ra[u], rp[u]);
  if (rest) {
    const f32x4v fz = {0.f, 0.f, 0.f, 0.f};
    const f32x4v x = xr[t_rest], p = pr[t_rest];
    use(rest_in ? x : fz, rest_in ? p : fz);
  }
  const double acc = (acc4[0] + acc4[1]) + (acc4[2] + acc4[3]);
  const double xx = (xx4[0] + xx4[1]) + (xx4[2] + xx4[3]);
  sh.part[wave][lane] = acc;
  sh.xx[wave][lane] = xx;
  __syncthreads();
  if (tid < 16 * PG) {
    const int m = tid & 3, pi = tid >> 2;  // token row of the tile, pivot of this group
    double d = 0.0, x2 = 0.0;
#pragma unroll
    for (int w = 0; w < kF32Waves; ++w) {
#pragma unroll
      for (int h = 0; h < kHalves; ++h) {
        d += sh.part[w][(pi & 3) + 4 * ((pi >> 2) + PG * h) + 16 * m];
#pragma unroll
        for (int k = 0; k < 4; ++k) x2 += sh.xx[w][m + 4 * (PG * h) + 16 * k];
      }
    }
    if (i0 + pi < P && j0 + m < n) {
      const double den = sqrt(pl2[b * g.Ppad + i0 + pi]) * sqrt(x2);
      Sb[(long)(i0 + pi) * n + j0 + m] = (float)(den > 0.0 ? d / den : 0.0) + 0.0f;
    }
  }
}

// Long rows, few of them (k_scores_f32_rows): two rows by 8 pivots at a time on the vector ALU.  A wave's
// load is 1 KiB of one row, where the matrix instructions want 4 or 16 rows side by side: from rows
// of 16 KiB on a compute unit takes in half again as much that way (about 50 against 31 GB/s), and with
// few pivots that counts for more than the arithmetic.  Scores of 1500 rows of 8192 by 8 pivots: 24.8 us,
// 31 on tiles of 16 rows or of 4; 576 rows by 8: 20, 23.  With more than 24 pivots it is always slower.
// Its 4 waves split D (piece t of a row goes to wave (t / 64) % 4); the next pieces are requested before
// the current ones are used; the 4 partial sums of a dot product are added in wave order, each wave's
// own sum is a fixed lane-strided order plus butterfly: a score depends only on the two rows' bytes.
constexpr int kF32Piv = 8, kF32Rows = 2;

// grid: tiles of 2 rows; 256 threads.
__global__ __launch_bounds__(256) void k_scores_f32_rows(Geo g, const void* __restrict__ X,
                                                         const int* __restrict__ piv,
                                                         const double* __restrict__ pl2,
                                                         float* __restrict__ S) {
  __shared__ double red[4][kF32Rows * kF32Piv + kF32Rows];  // per wave: dot[2][8], xx[2]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int b, tl;
  if (!locate_tile(g, blockIdx.x, b, tl)) return;
  const Sample sm = sample_of(g, b);
  const int n = sm.n, P = g.P, j0 = tl * kF32Rows;
  if (sm.k == 0 || j0 >= n) return;
  const float* Xb = static_cast<const float*>(X) + (long)sm.xrow * g.ld;
  const int pieces = g.D / 4;
  const f32x4v* xr[kF32Rows];
#pragma unroll
  for (int r = 0; r < kF32Rows; ++r) {
    const int j = j0 + r < n ? j0 + r : n - 1;  // rows past the end re-read the last; never stored
    xr[r] = reinterpret_cast<const f32x4v*>(Xb + (long)j * g.ld);
  }
  float* Sb = S + (long)P * sm.row0;
  const f32x4v fz = {0.f, 0.f, 0.f, 0.f};
  for (int i0 = 0; i0 < P; i0 += kF32Piv) {
    const f32x4v* pr[kF32Piv];
#pragma unroll
    for (int q = 0; q < kF32Piv; ++q) {
      const int i = i0 + q < P ? i0 + q : P - 1;
      pr[q] = reinterpret_cast<const f32x4v*>(pivot_row(g, X, 4, sm, b, i, piv));
    }
    double dot[kF32Rows][kF32Piv], xx[kF32Rows];
#pragma unroll
    for (int r = 0; r < kF32Rows; ++r) {
      xx[r] = 0.0;
#pragma unroll
      for (int q = 0; q < kF32Piv; ++q) dot[r][q] = 0.0;
    }
    f32x4v xv[kF32Rows], pv[kF32Piv], xn[kF32Rows], pn[kF32Piv];
    int t = tid;  // piece index: 256 apart per step
    auto fetch = [&](int tt, f32x4v (&xo)[kF32Rows], f32x4v (&po)[kF32Piv]) {
      const bool in = tt < pieces;
      const int ts = in ? tt : 0;  // a piece past the end re-reads piece 0 and counts as zero
#pragma unroll
      for (int r = 0; r < kF32Rows; ++r) {
        const f32x4v v = xr[r][ts];
        xo[r] = in ? v : fz;
      }
#pragma unroll
      for (int q = 0; q < kF32Piv; ++q) {
        const f32x4v v = pr[q][ts];
        po[q] = in ? v : fz;
      }
    };
    fetch(t, xv, pv);
    for (; t < pieces; t += 256) {
      fetch(t + 256, xn, pn);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        double x[kF32Rows];
#pragma unroll
        for (int r = 0; r < kF32Rows; ++r) {
          x[r] = (double)xv[r][e];
          xx[r] = fma(x[r], x[r], xx[r]);
        }
#pragma unroll
        for (int q = 0; q < kF32Piv; ++q) {
          const double p = (double)pv[q][e];
#pragma unroll
          for (int r = 0; r < kF32Rows; ++r) dot[r][q] = fma(p, x[r], dot[r][q]);
        }
      }
#pragma unroll
      for (int r = 0; r < kF32Rows; ++r) xv[r] = xn[r];
#pragma unroll
      for (int q = 0; q < kF32Piv; ++q) pv[q] = pn[q];
    }
    // the wave's sums, then the four waves' partials in wave order
#pragma unroll
    for (int r = 0; r < kF32Rows; ++r) {
#pragma unroll
      for (int q = 0; q < kF32Piv; ++q) {
        const double d = wave_sum(dot[r][q]);
        if (lane == 0) red[wave][r * kF32Piv + q] = d;
      }
      const double x2 = wave_sum(xx[r]);
      if (lane == 0) red[wave][kF32Rows * kF32Piv + r] = x2;
    }
    __syncthreads();
    if (tid < kF32Rows * kF32Piv) {
      const int r = tid / kF32Piv, q = tid - r * kF32Piv;
      if (i0 + q < P && j0 + r < n) {
        double d = 0.0, x2 = 0.0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          d += red[w][r * kF32Piv + q];
          x2 += red[w][kF32Rows * kF32Piv + r];
        }
        const double den = sqrt(pl2[b * g.Ppad + i0 + q]) * sqrt(x2);
        Sb[(long)(i0 + q) * n + j0 + r] = (float)(den > 0.0 ? d / den : 0.0) + 0.0f;
      }
    }
    __syncthreads();  // red is reused by the next group of pivots
  }
}

}  // namespace dart
