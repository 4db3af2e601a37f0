// Row L1 norms of the criterion tensor: the pivot criterion of DART (footnote of
// Section 3.3: the K-norm is an L1 norm; Table 1 caption: pivots have the largest
// norm).  One streaming pass over [rows, Dc]; HBM-bound.
#pragma once
#include "common.hpp"
#include "k_misc.hpp"

namespace dart {

// (fp32 sums of a piece: the one-launch kernel's)
// Sum of |x| over one 16-byte piece of bf16 values, as a fixed pairwise tree (3 roundings).
// |x| of a bf16 widened to fp32 is exact.
__device__ __forceinline__ float piece_abs_sum_bf16(const u32x4& v) {
  float a0 = fabsf(bf16_lo(v.x)) + fabsf(bf16_hi(v.x));
  float a1 = fabsf(bf16_lo(v.y)) + fabsf(bf16_hi(v.y));
  float a2 = fabsf(bf16_lo(v.z)) + fabsf(bf16_hi(v.z));
  float a3 = fabsf(bf16_lo(v.w)) + fabsf(bf16_hi(v.w));
  return (a0 + a1) + (a2 + a3);
}

// Sum of x^2 over one 16-byte piece of bf16 values: the squares are exact in fp32 (8-bit
// significands), the pairwise tree rounds three times (relative error <= 3 * 2^-24).
__device__ __forceinline__ float piece_sq_sum_bf16(const u32x4& v) {
  const float x0 = bf16_lo(v.x), x1 = bf16_hi(v.x), x2 = bf16_lo(v.y), x3 = bf16_hi(v.y);
  const float x4 = bf16_lo(v.z), x5 = bf16_hi(v.z), x6 = bf16_lo(v.w), x7 = bf16_hi(v.w);
  const float a0 = x0 * x0 + x1 * x1, a1 = x2 * x2 + x3 * x3;
  const float a2 = x4 * x4 + x5 * x5, a3 = x6 * x6 + x7 * x7;
  return (a0 + a1) + (a2 + a3);
}

// Relative bound on |fp32 norm - exact norm| for norms summed in fp32 (the one-launch kernel):
// piece tree, then one add per piece a lane owns, then the 6-step butterfly, each rounding at most
// 2^-24 relative on a sum of non-negative terms.
inline double l1_rel_bound_bf16(int Dc) {
  const int chain = (Dc / 8 + kWave - 1) / kWave;
  return (double)(3 + chain + 6 + 1) * 5.9604644775390625e-08;
}

// grid: ceil(rows / 4) blocks of 256 threads, rounded up to a multiple of 8; wave w of the grid
// (after xcd_contiguous) owns row w.  Lane l reads the pieces l, l+64, ... so a
// wave's loads are 1 KiB contiguous; 8 loads are in flight per lane.
// The sums run in fp64, in the order of row_l1_l2_f64 (a function of the row's bytes): pivot selection
// ranks by them without reading a row again, which was half of its time (selection of multi-crop 8.4
// us, 5.5 now, of video 13.5 and 6.9), and the pass has the vector ALU to spare: a row of 4096 takes some
// 1900 of the 2900 cycles in which the memory delivers one to every SIMD (the pass on multi-crop 32.6 us
// with fp32 sums, 33.9).  l1 gets the norms rounded to fp32.
// KEEP: ordinary loads, which leave the rows in the memory-side cache for the score
// kernel's second pass (worth it only if the whole matrix fits there); otherwise
// streaming (non-temporal) loads, which read faster.
// SPAN: the samples' rows are spans of C (Geo::span); packed row r belongs to the sample b
// with cu[b] <= r < cu[b+1] and lives at row span[b] + (r - cu[b]) of C.  Rows of a sample that
// is skipped are not read and their norms are left alone.
// PREP: the first 8 blocks are not for rows: block 0 fills the ragged offsets (prepare_body; this
// kernel needs none of them), which as a launch of its own takes 4-5 us before this one.
// L2SQ (when the rows are the hidden states themselves): also the squared Euclidean norm of every
// row, which the score kernel divides by and the pivots' norms are taken from.
template <int DT, bool KEEP, bool SPAN, bool L2SQ, bool PREP>
__global__ __launch_bounds__(256) void k_row_l1(const void* __restrict__ C, int Dc, long ldc,
                                                int rows, float* __restrict__ l1,
                                                double* __restrict__ l1d, Geo g,
                                                double* __restrict__ l2sq, PrepareArgs prep) {
  if (PREP && blockIdx.x < kXcds) {
    if (blockIdx.x == 0) prepare_body<256>(g, prep);
    return;
  }
  const unsigned bid = blockIdx.x - (PREP ? kXcds : 0), blocks = gridDim.x - (PREP ? kXcds : 0);
  const int lane = threadIdx.x & 63;
  // (ordinary loads: the plain order measured faster; streaming loads: a die per eighth)
  const long blk = KEEP ? (long)bid : xcd_contiguous(bid, blocks);
  const long row = blk * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int esz = DT == kBF16 ? 2 : 4;
  const int pieces = Dc * esz / 16;
  long crow = row;
  if (SPAN) {
    int lo = 0, hi = g.B;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (g.cu[mid] <= row) lo = mid; else hi = mid;
    }
    // (the offsets may be anything here: prepare_body checks them while this runs)
    const long at = row - g.cu[lo], n = (long)g.cu[lo + 1] - g.cu[lo], s0 = g.span[lo];
    if (at < 0 || at >= n || n > g.max_N || !sample_processed(g, (int)n) || s0 < 0 ||
        s0 + n > (long)g.x_rows)
      return;
    crow = s0 + at;
  }
  const u32x4* rp = reinterpret_cast<const u32x4*>(static_cast<const unsigned char*>(C) + crow * ldc * esz);
  double a = 0.0, b = 0.0;
  for (int t0 = 0; t0 < pieces; t0 += kWave * 8) {
    u32x4 v[8];
    load_pieces<8, !KEEP>(v, rp, t0, pieces, lane);
    add_pieces_l1_l2<DT, L2SQ>(v, t0, pieces, a, b);
  }
  a = wave_sum(a);
  if (L2SQ) b = wave_sum(b);
  if (lane == 0) {
    l1[row] = (float)a;
    l1d[row] = a;
    if (L2SQ) l2sq[row] = b;
  }
}

// Short rows (at most 64 pieces, criterion rows as a rule): R rows per wave, a load of each in flight,
// because the reduction and the wave's start cost more than such a row takes to read.
// The R sums are reduced together: lanes exchange half of their rows at every step, so that it takes
// R + 2 additions instead of 6 R, in the order of wave_sum: the same bits as row_l1_l2_f64, which sums
// such rows where the samples are spans or the norms the caller's.  PREP: as above.
template <int DT, int R, bool PREP>
__global__ __launch_bounds__(256) void k_short_row_l1(const void* __restrict__ C, int Dc, long ldc,
                                                      int rows, float* __restrict__ l1,
                                                      double* __restrict__ l1d, Geo g,
                                                      PrepareArgs prep) {
  static_assert(R == 8, "three halvings leave a row per eight lanes");
  if (PREP && blockIdx.x < kXcds) {
    if (blockIdx.x == 0) prepare_body<256>(g, prep);
    return;
  }
  const unsigned bid = blockIdx.x - (PREP ? kXcds : 0), blocks = gridDim.x - (PREP ? kXcds : 0);
  const int lane = threadIdx.x & 63;
  const long row0 = (xcd_contiguous(bid, blocks) * 4 + (threadIdx.x >> 6)) * R;
  if (row0 >= rows) return;
  const int esz = DT == kBF16 ? 2 : 4;
  const int pieces = Dc * esz / 16;
  const bool in = lane < pieces;
  u32x4 v[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const long row = row0 + r < rows ? row0 + r : rows - 1;
    v[r] = __builtin_nontemporal_load(
        reinterpret_cast<const u32x4*>(static_cast<const unsigned char*>(C) + row * ldc * esz) + (in ? lane : 0));
  }
  double a[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    double unused = 0.0;
    a[r] = 0.0;
    add_piece_l1_l2<DT, false>(v[r], a[r], unused);
    a[r] = in ? a[r] : 0.0;
  }
  // odd lanes go on with rows 4..7, then the lanes with bit 1 with the upper two, bit 2 the upper one
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    const double keep = lane & 1 ? a[4 + h] : a[h], give = lane & 1 ? a[h] : a[4 + h];
    a[h] = keep + lane_xor<1>(give, lane);
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const double keep = lane & 2 ? a[2 + h] : a[h], give = lane & 2 ? a[h] : a[2 + h];
    a[h] = keep + lane_xor<2>(give, lane);
  }
  const double keep = lane & 4 ? a[1] : a[0], give = lane & 4 ? a[0] : a[1];
  double s = keep + lane_xor<4>(give, lane);
  s += lane_xor<8>(s, lane);
  s += lane_xor<16>(s, lane);
  s += lane_xor<32>(s, lane);
  const long row = row0 + (lane & 1) * 4 + ((lane >> 1) & 1) * 2 + ((lane >> 2) & 1);
  if (lane < R && row < rows) {
    l1[row] = (float)s;
    l1d[row] = s;
  }
}

}  // namespace dart
