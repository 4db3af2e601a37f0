// Small kernels around the main passes: per-sample offsets for ragged batches,
// pivot norms for the stand-alone score entry point, and the row gather that
// compacts the retained tokens (the shortened sequence of Appendix D).
#pragma once
#include "common.hpp"

namespace dart {

// Ragged batches only.  One block of THREADS threads: validates the offsets and every
// sample and writes the packed offsets cu_keep[B+1] (retained rows; a skipped
// sample keeps 0) and tile_start[B+1] (score tiles of g.tile_rows rows).  status[0] becomes
// 1 if a non-empty sample was rejected (its sizes or budget, or a span that leaves X), 2 if
// cu_seqlens itself is not a non-decreasing sequence from 0 to total_N (then every sample
// is skipped).
// by_size (optional, B <= kMaxBySize): the samples ordered from the longest to the shortest
// (ties in batch order).  The ordering kernel runs one workgroup per compute unit, a list's
// time grows with its sample's length, and workgroups start in id order: with the long
// samples first the short ones fill the gaps at the end instead of the other way round.
// seq_cu (optional, spans only): sequence b is rows [seq_cu[b], seq_cu[b+1]) of the caller's
// per-token tensors and must contain its span [span[b], span[b] + N_b).  seq_cu_out[B+1] gets the
// new offsets: sequence b shrinks by N_b - K_b rows (K_b = 0 for a skipped sample, whose vision
// tokens are all dropped).  status[2] = 1 and all-zero offsets if seq_cu is not a non-decreasing
// sequence from 0 to x_rows, a span is not inside its sequence, or cu_seqlens is broken.
struct PrepareArgs {
  int* cu_keep;
  int* tile_start;
  int* status;
  int* by_size;
  const int* seq_cu;
  int* seq_cu_out;
};

template <int THREADS>
__device__ __forceinline__ void prepare_body(const Geo& g, const PrepareArgs& a) {
  constexpr int kWaves = THREADS / kWave;
  __shared__ int red[3][kWaves];
  __shared__ int carry[3];
  __shared__ int len_of[kMaxBySize];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  int broken = 0, seq_bad = 0;
  for (int b = tid; b < g.B; b += THREADS) {
    const int n = g.cu[b + 1] - g.cu[b];
    broken |= n < 0 ? 1 : 0;
    if (a.seq_cu) {
      const int lo = a.seq_cu[b], hi = a.seq_cu[b + 1];
      seq_bad |= (hi < lo || g.span[b] < lo || (long)g.span[b] + n > (long)hi) ? 1 : 0;
    }
  }
  if (tid == 0) {
    carry[0] = carry[1] = carry[2] = 0;
    broken |= (g.cu[0] != 0 || g.cu[g.B] != g.total_N) ? 1 : 0;
    if (a.seq_cu) seq_bad |= (a.seq_cu[0] != 0 || a.seq_cu[g.B] != g.x_rows) ? 1 : 0;
  }
  broken = __syncthreads_or(broken);
  if (a.seq_cu) seq_bad = __syncthreads_or(seq_bad) | broken;  // (broken: the lengths are meaningless)
  int bad = 0;
  for (int b0 = 0; b0 < g.B; b0 += THREADS) {
    const int b = b0 + tid;
    int k = 0, tiles = 0, rows = 0;
    if (b < g.B && !broken) {
      int n = g.cu[b + 1] - g.cu[b];
      int kb = budget_of(g, n);
      // a span must lie inside X (long arithmetic: the caller's start may be anything)
      const bool inside = g.span == nullptr ||
                          (g.span[b] >= 0 && (long)g.span[b] + n <= (long)g.x_rows);
      if (inside && sample_ok(g, n, kb)) {
        k = kb;
        tiles = (n + g.tile_rows - 1) / g.tile_rows;
      } else if (n != 0) {
        bad = 1;
      }
      if (a.seq_cu && !seq_bad) rows = (a.seq_cu[b + 1] - a.seq_cu[b]) - n + k;
    }
    const int s[3] = {wave_excl_scan(k, lane), wave_excl_scan(tiles, lane), wave_excl_scan(rows, lane)};
    if (lane == 63) {
      red[0][w] = s[0] + k;
      red[1][w] = s[1] + tiles;
      red[2][w] = s[2] + rows;
    }
    __syncthreads();
    int base[3], sum[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      base[q] = carry[q];
      sum[q] = 0;
#pragma unroll
      for (int i = 0; i < kWaves; ++i) {
        base[q] += i < w ? red[q][i] : 0;
        sum[q] += red[q][i];
      }
    }
    if (b < g.B) {
      a.cu_keep[b] = base[0] + s[0];
      a.tile_start[b] = base[1] + s[1];
      if (a.seq_cu) a.seq_cu_out[b] = base[2] + s[2];
    }
    __syncthreads();
    if (tid < 3) carry[tid] += tid == 0 ? sum[0] : tid == 1 ? sum[1] : sum[2];
    __syncthreads();
  }
  bad = __syncthreads_or(bad);
  if (a.by_size != nullptr) {  // (block-uniform; g.B <= kMaxBySize)
    for (int b = tid; b < g.B; b += THREADS) len_of[b] = broken ? 0 : g.cu[b + 1] - g.cu[b];
    __syncthreads();
    for (int b = tid; b < g.B; b += THREADS) {
      const int n = len_of[b];
      int rank = 0;
      for (int o = 0; o < g.B; ++o) rank += (len_of[o] > n || (len_of[o] == n && o < b)) ? 1 : 0;
      a.by_size[rank] = b;
    }
  }
  if (tid == 0) {
    a.cu_keep[g.B] = carry[0];
    a.tile_start[g.B] = carry[1];
    if (a.seq_cu) a.seq_cu_out[g.B] = carry[2];
    a.status[0] = broken ? 2 : bad;
    a.status[2] = a.seq_cu ? seq_bad : 0;
  }
}

__global__ __launch_bounds__(1024) void k_prepare(Geo g, PrepareArgs a) { prepare_body<1024>(g, a); }

// Caller-supplied pivots: status[1] = 1 if any processed sample's Pin indices are not
// distinct indices inside the sample, else 0.  grid: 1 block of 1024.
__global__ __launch_bounds__(1024) void k_check_pivots(Geo g, const int* __restrict__ piv,
                                                       int* __restrict__ status) {
  int bad = 0;
  for (int idx = threadIdx.x; idx < g.B * g.P; idx += 1024) {
    const int b = idx / g.P, i = idx - b * g.P;
    if (i >= g.Pin) continue;  // a pivot from outside the sample: nothing to check
    const Sample sm = sample_of(g, b);
    if (sm.k == 0) continue;
    const int p = piv[idx];
    bad |= (p < 0 || p >= sm.n) ? 1 : 0;
    for (int o = 0; o < i; ++o) bad |= piv[b * g.P + o] == p ? 1 : 0;
  }
  bad = __syncthreads_or(bad);
  if (threadIdx.x == 0) status[1] = bad ? 1 : 0;
}

// Pivots drawn at random (the random rows of the pivot ablation, Section 4.3 / Table 8).
// The generator is Philox4x32 with 10 rounds (Salmon, Moraes, Dror, Shaw, SC'11): a round maps
// the counter words (c0, c1, c2, c3) to (hi(M1 c2) ^ c1 ^ k0, lo(M1 c2), hi(M0 c0) ^ c3 ^ k1,
// lo(M0 c0)); the key words grow by the two Weyl constants between rounds.
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t (&out)[4]) {
  constexpr uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u;
#pragma unroll
  for (int round = 0; round < 10; ++round) {
    if (round > 0) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
    }
    const uint32_t hi0 = __umulhi(M0, c0), lo0 = M0 * c0;
    const uint32_t hi1 = __umulhi(M1, c2), lo1 = M1 * c2;
    c0 = hi1 ^ c1 ^ k0;
    c1 = lo1;
    c2 = hi0 ^ c3 ^ k1;
    c3 = lo0;
  }
  out[0] = c0;
  out[1] = c1;
  out[2] = c2;
  out[3] = c3;
}

// Sample b draws tokens d_t = floor(w_t * N_b / 2^32), t = 0, 1, ..., with w_t word t mod 4 of
// the Philox block of counter (t div 4, b, 0, 0) and key (low, high half of the seed); its
// Pin pivots are the first Pin distinct draws in the order they appear.  After draw_limit
// draws (kRandomDraws, a bound for the loop: 64 pivots among 64 tokens need about 300; a test
// may lower it) the lowest unused tokens fill the list.  grid: B blocks of one wave: the lanes
// compute 256 draws at a time, lane 0 walks them.
constexpr int kRandomDraws = 4096;
__global__ __launch_bounds__(64) void k_random_pivots(Geo g, unsigned long long seed,
                                                      int draw_limit, int* __restrict__ piv) {
  __shared__ uint32_t used[kMaxN / 32];
  __shared__ int draws[256];
  __shared__ int have_sh;
  const int b = blockIdx.x, lane = threadIdx.x;
  const Sample sm = sample_of(g, b);
  if (sm.k == 0 || g.Pin == 0) return;
  const int n = sm.n, want = g.Pin;
  int* out = piv + (long)b * g.P;
  for (int t = lane; t < (n + 31) / 32; t += 64) used[t] = 0u;
  int have = 0;
  for (int base = 0; base < draw_limit && have < want; base += 256) {
    uint32_t w[4];
    philox4x32_10((uint32_t)(base / 4 + lane), (uint32_t)b, 0u, 0u, (uint32_t)seed,
                  (uint32_t)(seed >> 32), w);
#pragma unroll
    for (int u = 0; u < 4; ++u) draws[4 * lane + u] = (int)__umulhi(w[u], (uint32_t)n);
    __syncthreads();
    if (lane == 0) {
      for (int t = 0; t < 256 && base + t < draw_limit && have < want; ++t) {
        const int d = draws[t];
        const uint32_t bit = 1u << (d & 31);
        if ((used[d >> 5] & bit) == 0u) {
          used[d >> 5] |= bit;
          out[have++] = d;
        }
      }
      have_sh = have;
    }
    __syncthreads();
    have = have_sh;
  }
  if (lane == 0)
    for (int j = 0; j < n && have < want; ++j)
      if ((used[j >> 5] & (1u << (j & 31))) == 0u) out[have++] = j;
}

// status[1] = 0: for entry points that read no pivot list (one thread).
__global__ void k_clear_pivot_status(int* __restrict__ status) { status[1] = 0; }

// The raw matrix-core sums the bf16 score kernel is built on, for the test of its rounding
// bound: tile t of A and B is [16][32] bf16 (k contiguous); out[t][i][j] = sum_k A[i][k] *
// B[j][k] from a zero accumulator.  grid: tiles blocks of 64.
typedef __bf16 probe_bf16x8 __attribute__((ext_vector_type(8)));
typedef float probe_f32x4 __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(64) void k_probe_mfma_dot32(const unsigned char* __restrict__ A,
                                                        const unsigned char* __restrict__ B,
                                                        float* __restrict__ out) {
  const int lane = threadIdx.x;
  const long tile = blockIdx.x;
  const long off = tile * (16 * 32 * 2) + (lane & 15) * 64 + (lane >> 4) * 16;
  const probe_bf16x8 af = *reinterpret_cast<const probe_bf16x8*>(A + off);
  const probe_bf16x8 bf = *reinterpret_cast<const probe_bf16x8*>(B + off);
  const probe_f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  const probe_f32x4 c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bf, zero, 0, 0, 0);
#pragma unroll
  for (int r = 0; r < 4; ++r) out[tile * 256 + ((lane >> 4) * 4 + r) * 16 + (lane & 15)] = c[r];
}

// Squared Euclidean norms of the rows of the pivots in fp64 (0 for padding
// slots).  piv_mark (optional): entry i of a pivot from outside the sample is set to
// -1 - (its row in the sample's share of E).  grid: B blocks of 1024: a wave per pivot, so
// that up to 16 rows are in flight at once (64 pivots: four rounds).
template <int DT>
__global__ __launch_bounds__(1024) void k_pivot_norms(Geo g, const void* __restrict__ X,
                                                     const int* __restrict__ piv,
                                                     double* __restrict__ pl2,
                                                     int* __restrict__ piv_mark) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b = blockIdx.x;
  const Sample sm = sample_of(g, b);
  const int esz = DT == kBF16 ? 2 : 4;
  if (piv_mark && tid >= g.Pin && tid < g.P) piv_mark[b * g.P + tid] = -1 - (tid - g.Pin);
  for (int i = wave; i < g.Ppad; i += 16) {
    double l1 = 0.0, l2 = 0.0;
    if (sm.k != 0 && i < g.P) row_l1_l2_f64<DT>(pivot_row(g, X, esz, sm, b, i, piv), g.D, lane, l1, l2);
    if (lane == 0) pl2[b * g.Ppad + i] = l2;
  }
}

// A row by one wave: 16 bytes per lane, 1 KiB per access, eight accesses in flight.
__device__ __forceinline__ void copy_row(const u32x4* in, u32x4* out, int pieces, int lane) {
  for (int t0 = 0; t0 < pieces; t0 += kWave * 8) {
    u32x4 v[8];
    load_pieces<8, true>(v, in, t0, pieces, lane);
    if (t0 + 8 * kWave <= pieces) {
#pragma unroll
      for (int u = 0; u < 8; ++u) out[t0 + u * kWave + lane] = v[u];
    } else {
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int t = t0 + u * kWave + lane;
        if (t < pieces) out[t] = v[u];
      }
    }
  }
}

// Compaction: one wave per retained row.  grid: ceil(rows_bound / 4) blocks of 256, rounded up
// to a multiple of 8 (xcd_contiguous).
// Y rows are packed (stride D); copies are 16 bytes per lane, 1 KiB per wave access.
// The rows are read once: streaming (non-temporal) loads measured 20 % faster on the
// largest batch than ordinary ones; streaming stores did not help.
__global__ __launch_bounds__(256) void k_gather(Geo g, int esz, const void* __restrict__ X,
                                                const long long* __restrict__ pos,
                                                const int* __restrict__ keep,
                                                void* __restrict__ Y,
                                                long long* __restrict__ pos_out) {
  const int lane = threadIdx.x & 63;
  const long r = xcd_contiguous(blockIdx.x, gridDim.x) * 4 +
                 __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int b;
  if (g.cu == nullptr) {
    if (r >= (long)g.B * g.K) return;
    b = (int)(r / g.K);
  } else {
    if (r >= g.cu_keep[g.B]) return;
    b = -1;
  }
  int kr = keep[r];  // (requested ahead of the search)
  if (b < 0) b = last_at_most(g.cu_keep, g.B, (int)r);
  const int row0 = g.cu ? g.cu[b] : b * g.N;
  const int n = g.cu ? g.cu[b + 1] - row0 : g.N;
  kr = kr < 0 ? 0 : (kr < n ? kr : n - 1);  // a caller's bad index must not leave X
  const long src = (long)(g.span ? g.span[b] : row0) + kr;
  const u32x4* in = reinterpret_cast<const u32x4*>(static_cast<const unsigned char*>(X) +
                                                   src * g.ld * esz);
  u32x4* out = reinterpret_cast<u32x4*>(static_cast<unsigned char*>(Y) + r * (long)g.D * esz);
  const int pieces = g.D * esz / 16;
  copy_row(in, out, pieces, lane);
  if (pos && lane == 0) pos_out[r] = pos[src];
}

// ---- whole-sequence compaction (Appendix D: text before the vision span, the retained
// vision tokens, text after it) ------------------------------------------------------

constexpr int kSeqOps = 8;  // tensors one gather launch moves
struct SeqOps {
  const unsigned char* src[kSeqOps];
  unsigned char* dst[kSeqOps];
  long row_bytes[kSeqOps], src_ld[kSeqOps], dst_ld[kSeqOps];  // bytes, multiples of 16
};
struct SeqPos {  // position ids, plane-major
  const long long* pos;
  long long* pos_out;
  long in_stride, out_stride;
  int planes;
};

// Row r of the shortened batch comes from row src(r) of the original tensors: the rows of its
// sequence before the span, then span + keep, then the rows behind the span.
struct SeqRow {  // the sample of a row: the last one whose new offset is at most r
  int off, end;  // its rows are [off, end) of the shortened batch
  int s0, span, n, k0, k;
  __device__ __forceinline__ void load(const Geo& g, const int* seq_cu, const int* seq_cu_out, int b) {
    off = seq_cu_out[b];
    end = seq_cu_out[b + 1];
    s0 = seq_cu[b];
    span = g.span[b];
    n = g.cu[b + 1] - g.cu[b];
    k0 = g.cu_keep[b];
    k = g.cu_keep[b + 1] - k0;
  }
  __device__ __forceinline__ long source(int r, const int* keep) const {
    const int t = r - off, before = span - s0;  // text rows ahead of the span
    if (t < before) return s0 + t;
    if (t >= before + k) return span + n + (t - before - k);
    int kr = keep[k0 + (t - before)];
    kr = kr < 0 ? 0 : (kr < n ? kr : n - 1);  // a caller's bad index must not leave the span
    return span + kr;
  }
};

// The map and the position planes, a row per thread, where there are no tensors to move or many
// sequences (see k_gather_rows).  grid: ceil(rows_bound / 256) blocks of 256.  (590 000 rows of 16384
// sequences, the offsets' launch included: 62 us; 85 at best with the rows dealt as in k_gather_rows.)
__global__ __launch_bounds__(256) void k_seq_row_map(Geo g, const int* __restrict__ seq_cu,
                                                     const int* __restrict__ seq_cu_out,
                                                     const int* __restrict__ keep,
                                                     int* __restrict__ row_map, SeqPos sp) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= seq_cu_out[g.B]) return;
  int lo = 0, hi = g.B;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (seq_cu_out[mid] <= r) lo = mid; else hi = mid;
  }
  SeqRow q;
  q.load(g, seq_cu, seq_cu_out, lo);
  const long src = q.source(r, keep);
  row_map[r] = (int)src;
  for (int p = 0; p < sp.planes; ++p)
    sp.pos_out[p * sp.out_stride + r] = sp.pos[p * sp.in_stride + src];
}

// dst row r = src row src(r) for every tensor of ops.  Every wave works out its rows' sources by
// itself, so that the map, the position ids and the tensors need one launch (five launches of which
// three moved a few KB took 38 us on eight sequences of 1900 rows, two take 28); the waves of
// tensor 0 also write row_map and the position planes (first: the first launch of the call).
// A row's sample is found by 64 offsets in the lanes and a ballot; of more samples every look leaves
// a 64th (one after the other, 64 at a time, 4096 sequences of 20 tokens and nine tensors of 512
// bytes took 2875 us; 281 now, 351 with a launch for the map before it).
// A wave per R rows of a tensor: grid (ceil(rows_bound / (4 R)) rounded up to a multiple of 8, tensors)
// blocks of 256 (with a multiple of 8 in x the die of a block depends on its x only: xcd_contiguous);
// 16 bytes per lane, 1 KiB per access.  R > 1 (rows of at most 2 KiB): what a wave has to find out
// takes longer than a short row takes to move, and several rows are in flight together.  R rows
// per wave: 1, 2, 4, 8, 16, by 64 sequences of 937 tokens and nine tensors of 512 bytes: 58, 41, 36,
// 39, 44 us; rows of 1 KiB, 4096 sequences of 20 tokens: 97, 69, 64, 67, 71; of 2 KiB: 131, 126, 124,
// 127, 125, but eight tensors of 2 KiB in 64 sequences 74, 75, 76, 84, 88; of 8 KiB, five tensors: 236,
// -, 255, 269, -.  Rows beyond seq_cu_out[B] are left alone.
// MAPPED: k_seq_row_map has written the map and the positions.  Of more than kSeqMapped sequences with
// rows of over 1 KiB: looking the sample up costs such batches more than that launch (four tensors of
// 2080 bytes, 1000 sequences of 60 tokens 149 us, 155 without; 500 of 120 tokens 87 without, 83 before
// the map and the gather were one launch; 300 of 200 tokens 66 without, 70 then).
constexpr int kSeqMapped = 384;
template <int R, bool MAPPED>
__global__ __launch_bounds__(256) void k_gather_rows(Geo g, SeqOps ops, bool first,
                                                     const int* __restrict__ seq_cu,
                                                     const int* __restrict__ seq_cu_out,
                                                     const int* __restrict__ keep,
                                                     int* __restrict__ row_map, SeqPos sp) {
  const int lane = threadIdx.x & 63, o = blockIdx.y;
  const int r0 = __builtin_amdgcn_readfirstlane(
      (int)(xcd_contiguous(blockIdx.x, gridDim.x) * 4 + (threadIdx.x >> 6)) * R);
  const int rows = seq_cu_out[g.B];
  if (r0 >= rows) return;
  SeqRow q;
  q.end = 0;
  auto find = [&](int r) { q.load(g, seq_cu, seq_cu_out, last_at_most(seq_cu_out, g.B, r)); };
  long src[R];
#pragma unroll
  for (int u = 0; u < R; ++u) {
    src[u] = 0;
    if (r0 + u >= rows) continue;
    if (MAPPED) {
      src[u] = row_map[r0 + u];
      continue;
    }
    if (r0 + u >= q.end) find(r0 + u);
    src[u] = q.source(r0 + u, keep);
  }
  if (!MAPPED && o == 0 && first) {
    const int u = lane % R;
    long mine = src[0];
#pragma unroll
    for (int v = 1; v < R; ++v) mine = u == v ? src[v] : mine;
    if (r0 + u < rows) {
      if (lane < R) row_map[r0 + u] = (int)mine;
      for (int p = lane / R; p < sp.planes; p += kWave / R)
        sp.pos_out[p * sp.out_stride + r0 + u] = sp.pos[p * sp.in_stride + mine];
    }
  }
  const u32x4 zero = {0u, 0u, 0u, 0u};
  const int pieces = (int)(ops.row_bytes[o] / 16);
  auto row_in = [&](int u) { return reinterpret_cast<const u32x4*>(ops.src[o] + src[u] * ops.src_ld[o]); };
  auto row_out = [&](int u) { return reinterpret_cast<u32x4*>(ops.dst[o] + (long)(r0 + u) * ops.dst_ld[o]); };
  if (R > 1) {  // (pieces <= 2 * kWave: see the launch) all rows in flight
    u32x4 v[R][2];
#pragma unroll
    for (int u = 0; u < R; ++u)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int t = h * kWave + lane;
        v[u][h] = r0 + u < rows && t < pieces ? __builtin_nontemporal_load(row_in(u) + t) : zero;
      }
#pragma unroll
    for (int u = 0; u < R; ++u)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int t = h * kWave + lane;
        if (r0 + u < rows && t < pieces) row_out(u)[t] = v[u][h];
      }
    return;
  }
  copy_row(row_in(0), row_out(0), pieces, lane);
}

}  // namespace dart
