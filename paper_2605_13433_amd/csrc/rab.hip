// Standalone relative attention bias (RAB) of Sec. 4.1.1's operator on
// gfx950: the jagged bias tensor (one L x L square per sequence, no
// padding) from the position table, the bucketed time table and a
// functional time encoding, and its backward into those parameters.
//
// Both passes cut the batch into equal wave items, numbered across the
// sequences (rab_scan_kernel's prefix sums): a 2048-token sequence's square is
// spread as evenly as a hundred short ones.
//
// Forward, bound by its writes: an item is 512 consecutive elements of a
// square, whatever rows they belong to, for every head.  The time bucket,
// log2(1 + |dt|) and position index of an element belong to its pair of rows,
// not to a head, and are computed once.  Consecutive elements, because a
// wave that writes 256-byte pieces of many unaligned rows leaves the 128-byte
// lines at their ends to other waves: 3.3 TB/s for the bare stores of
// 16 x 64 tiles, 4.6 TB/s for runs, 5.5 TB/s where all planes are aligned.
// One eighth of the items go to each XCD, so that shared lines meet in one L2
// (another 8% for the tiles).
//
// Backward, bound by its reads and the per-element double sums: sheared
// items of 32 rows by 64 diagonals, lane l on diagonal d0 + l.  In any row the
// lanes read 64 consecutive columns, and down the rows a lane stays on its
// diagonal, so the position gradient is a plain sum in a register.  Two heads
// share a work-group (and an element's bucket and logarithm); it keeps their
// time histograms in LDS, one 64-bit fixed-point counter per bucket and lane
// group, added to at the end of each run of equal buckets down a diagonal.
// Lanes on neighbouring diagonals meet in the same bucket and a wave's
// atomics on one address are served one by one, so four heads (16 counters
// per bucket) took 1010 us where two (32) take 257 and one (64) 356.  The
// functional encoding's sums stay in registers.  All partial sums are in
// double; what crosses waves is 64-bit fixed point added with integer
// atomics, or a sum in a fixed order: the result does not depend on the
// order in which work-groups finish, so the backward is bitwise reproducible.
//
// Measured on 64 sequences of 32..2048 tokens, 8 heads (841 MB), all three
// encodings: forward 1630 -> 182 us (4.6 TB/s), backward 2480 -> 257 us
// (3.3 TB/s; reading alone, position gradient only, 189 us).  Before, one
// work-group walked a 64-row band per head, which computed every bucket and
// logarithm per head and left the longest bands to the end.
#include <algorithm>

#include "internal.h"
#include "device.h"

namespace hstu {
namespace {

constexpr int R_ROWS = 32;                   // rows of an item
constexpr int R_STEP = 8;                    // rows handled at a time (16 spills)
constexpr int R_FSTEP = 8;                   // elements of a lane in a forward item
constexpr int R_FLAT = 64 * R_FSTEP;         // consecutive elements of a forward item
constexpr int R_FWD_THREADS = 256;
constexpr int R_BWD_THREADS = 512;
constexpr int R_SCAN_THREADS = 1024;
// Item prefix in LDS up to this many sequences (read from L2 above).
constexpr int R_LDS_SEQS = 1023;
// LDS counters of the backward's time histograms (64 KB, two work-groups per
// CU): with two heads 32 per bucket up to 128 buckets, fewer above.
constexpr int R_HIST = 8192;
constexpr int64_t R_NEAR = 1 << 30;          // gaps of timestamps this near fit 32 bits

struct RabArgs {
  const int64_t *off;
  int64_t *sq;                          // [B+1] square offsets (workspace)
  int64_t *items;                       // [B+1] item offsets (workspace)
  const float *pos_w, *time_w, *time_fn;
  const int64_t *ts;
  float *rab;
  const float *d_rab;
  // table sums, back to back in the workspace (n_fix in all)
  unsigned long long *fix, *fix_pos, *fix_time, *fix_fn;
  int64_t n_fix;
  int64_t T, total_square;
  int B, N, H, nb;
  int copies;                           // histogram counters per bucket
};

// Clamped start and length of sequence b (as the attention's scheduler
// clamps them: every row index stays inside [0, T)).
__device__ __forceinline__ void seq_of(const RabArgs &a, int b, int64_t &start, int &len) {
  int64_t s0 = a.off[b], s1 = a.off[b + 1];
  s0 = s0 < 0 ? 0 : (s0 > a.T ? a.T : s0);
  s1 = s1 < s0 ? s0 : (s1 > a.T ? a.T : s1);
  int64_t L = s1 - s0;
  start = s0;
  len = (int)(L > a.N ? a.N : L);
}

// 64-diagonal strips that cover `rows` rows of a square of side L, and the
// items of the whole square (`flat`: the forward's, else the backward's).
__device__ __forceinline__ int strips_of(int L, int rows) { return (L + rows - 1 + 63) / 64; }
__device__ __forceinline__ int64_t items_of(int L, bool flat) {
  if (flat) return ((int64_t)L * L + R_FLAT - 1) / R_FLAT;
  const int full = L / R_ROWS, rem = L % R_ROWS;
  return (int64_t)full * strips_of(L, R_ROWS) + (rem ? strips_of(L, rem) : 0);
}

// sq[b] = sum of L_b'^2 and items[b] = sum of items over b' < b (work-group
// 0: a wave scan of each 1024 sequences); the other work-groups clear the
// backward's table sums.
__global__ void __launch_bounds__(R_SCAN_THREADS) rab_scan_kernel(RabArgs a) {
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  if (blockIdx.x > 0) {
    for (int64_t x = (int64_t)(blockIdx.x - 1) * R_SCAN_THREADS + t; x < a.n_fix;
         x += (int64_t)(gridDim.x - 1) * R_SCAN_THREADS)
      a.fix[x] = 0;
    return;
  }
  constexpr int W = R_SCAN_THREADS / 64;
  __shared__ int64_t part[2][W];
  int64_t run_s = 0, run_i = 0;
  for (int b0 = 0; b0 < a.B; b0 += R_SCAN_THREADS) {
    const int b = b0 + t;
    int64_t st, sq = 0, it = 0;
    if (b < a.B) {
      int L;
      seq_of(a, b, st, L);
      sq = (int64_t)L * L;
      it = items_of(L, a.rab != nullptr);
    }
    int64_t s = sq, n = it;                       // inclusive sums over the wave
#pragma unroll
    for (int k = 1; k < 64; k <<= 1) {
      const int64_t us = __shfl_up(s, k, 64), un = __shfl_up(n, k, 64);
      s += lane >= k ? us : 0;
      n += lane >= k ? un : 0;
    }
    __syncthreads();
    if (lane == 63) { part[0][w] = s; part[1][w] = n; }
    __syncthreads();
    int64_t before_s = run_s, before_i = run_i;
    for (int x = 0; x < W; ++x) {
      if (x < w) { before_s += part[0][x]; before_i += part[1][x]; }
      run_s += part[0][x];
      run_i += part[1][x];
    }
    if (b < a.B) {
      a.sq[b] = before_s + s - sq;
      a.items[b] = before_i + n - it;
    }
  }
  if (t == 0) { a.sq[a.B] = run_s; a.items[a.B] = run_i; }
}

// 64-bit fixed-point value of a double partial sum (as to_fix).
__device__ __forceinline__ unsigned long long fix_d(double v) {
  return (unsigned long long)(long long)__builtin_rint(v * FIX_ONE);
}

// log2(1 + |dt|) of the functional time term g = (1 + |dt|)^(-beta)
// (32-bit conversion while |dt| fits, the common case).
__device__ __forceinline__ float fn_lg2(int64_t dt) {
  const uint64_t x = dt < 0 ? (uint64_t)0 - (uint64_t)dt : (uint64_t)dt;
  const float xf = x < (1u << 31) ? (float)(uint32_t)x : (float)x;
  return __builtin_amdgcn_logf(1.0f + xf);
}

// The item prefix where a work-group finds it: staged in LDS, or (many
// sequences) in the workspace.
__device__ __forceinline__ const int64_t *stage_items(const RabArgs &a, int64_t *lds, int tid,
                                                      int threads) {
  if (a.B > R_LDS_SEQS) return a.items;
  for (int b = tid; b <= a.B; b += threads) lds[b] = a.items[b];
  __syncthreads();
  return lds;
}

// Sequence of item `item`: the last one whose items begin at or before it
// (the same in every lane).
__device__ __forceinline__ int seq_of_item(const RabArgs &a, const int64_t *items, int64_t item) {
  int lo = 0, hi = a.B - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (items[mid] <= item) lo = mid; else hi = mid - 1;
  }
  return __builtin_amdgcn_readfirstlane(lo);
}

// Wave item `item`: rows r0 .. r0 + rows - 1 of the sequence at `start`, whose
// square of side L begins at element `base`; lane l is on diagonal (column
// minus row) d0 + l.  All wave-uniform.
struct Strip {
  int64_t start, base;
  int L, r0, rows, d0;
};

// False if the square would not fit the caller's tensor.
__device__ __forceinline__ bool strip_of(const RabArgs &a, const int64_t *items, int64_t item,
                                         Strip &t) {
  const int b = seq_of_item(a, items, item);
  seq_of(a, b, t.start, t.L);
  t.base = a.sq[b];
  const int local = __builtin_amdgcn_readfirstlane((int)(item - items[b]));
  const int full = t.L / R_ROWS, ns = strips_of(t.L, R_ROWS);
  int rc = local / ns;
  rc = rc < full ? rc : full;
  t.r0 = rc * R_ROWS;
  t.rows = t.L - t.r0 < R_ROWS ? t.L - t.r0 : R_ROWS;
  t.d0 = 64 * (local - rc * ns) - (t.r0 + t.rows - 1);
  return t.base >= 0 && t.base + (int64_t)t.L * t.L <= a.total_square;
}

// Rows k0 .. k0 + R_STEP - 1 of a strip for a lane on diagonal d: bit k set
// where row k0 + k exists and its column lies in the square.
__device__ __forceinline__ uint32_t step_ok(const Strip &t, int k0, int d) {
  const int i0 = t.r0 + k0;
  int lo = -(i0 + d), hi = t.L - (i0 + d);                 // columns 0 .. L - 1
  lo = lo < 0 ? 0 : (lo > R_STEP ? R_STEP : lo);
  const int left = t.rows - k0 < R_STEP ? t.rows - k0 : R_STEP;
  hi = hi < 0 ? 0 : (hi > left ? left : hi);
  return hi > lo ? ((1u << hi) - 1u) & ~((1u << lo) - 1u) : 0u;
}

// log2(1 + y) of a 32-bit gap.
__device__ __forceinline__ float fn_lg2_32(uint32_t y) {
  return __builtin_amdgcn_logf(1.0f + (float)y);
}

// What the heads share of R_STEP rows from k0 on: time bucket and
// log2(1 + |dt|) of this lane's elements.  `near`: the strip's timestamps lie
// within 2^30 of the sequence's first, and `cols` (LDS) and `row` (lane k: row
// k) hold the differences; else the 64-bit rule on the timestamps themselves.
template <bool TIME, bool FN>
__device__ __forceinline__ void step_keys(const RabArgs &a, const Strip &t, int k0, int lane,
                                          bool near, const int32_t *cols, int32_t row,
                                          int (&bk)[R_STEP], float (&l2)[R_STEP]) {
  if (near) {
#pragma unroll
    for (int k = 0; k < R_STEP; ++k) {
      const int32_t ri = __builtin_amdgcn_readlane(row, k0 + k), cj = cols[k0 + k + lane];
      const uint32_t y = ri > cj ? (uint32_t)(ri - cj) : (uint32_t)(cj - ri);
      if (TIME) bk[k] = time_bucket_u32(y, a.nb);
      if (FN) l2[k] = fn_lg2_32(y);
    }
  } else {
#pragma unroll 1
    for (int k = 0; k < R_STEP; ++k) {
      const int i = t.r0 + k0 + k, j = i + t.d0 + lane;
      const int64_t *ts = a.ts + t.start;
      const int64_t dt = ts[i < t.L ? i : t.L - 1] - ts[j < 0 ? 0 : (j < t.L ? j : t.L - 1)];
      const int bv = TIME ? time_bucket32(dt, a.nb) : 0;
      const float lv = FN ? fn_lg2(dt) : 0.0f;
#pragma unroll
      for (int x = 0; x < R_STEP; ++x) {
        if (TIME) bk[x] = x == k ? bv : bk[x];
        if (FN) l2[x] = x == k ? lv : l2[x];
      }
    }
  }
}

// Dynamic LDS: every head's time table ([H][nb]) when time_w is given.
template <bool POS, bool TIME, bool FN>
__global__ void __launch_bounds__(R_FWD_THREADS) rab_fwd_kernel(RabArgs a) {
  __shared__ int64_t s_items[R_LDS_SEQS + 1];
  extern __shared__ float ttab[];
  constexpr int WAVES = R_FWD_THREADS / 64;
  const int tid = threadIdx.x, lane = tid & 63;
  if (TIME)
    for (int x = tid; x < a.H * a.nb; x += R_FWD_THREADS) ttab[x] = a.time_w[x];
  const int64_t *items = stage_items(a, s_items, tid, R_FWD_THREADS);
  if (TIME) __syncthreads();
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t n_items = items[a.B], span = 2 * (int64_t)a.N - 1;
  // one eighth of the items to each XCD (work-group i runs on XCD i % 8), so
  // that the lines neighbouring items share are completed in one L2
  const int64_t share = (n_items + 8 * WAVES - 1) / (8 * WAVES) * WAVES;
  const int64_t first = (blockIdx.x & 7) * share;
  const int64_t end = first + share < n_items ? first + share : n_items;
  for (int64_t item = first + (int64_t)(blockIdx.x >> 3) * WAVES + w; item < end;
       item += (int64_t)(gridDim.x >> 3) * WAVES) {
    const int b = seq_of_item(a, items, item);
    int64_t start;
    int L;
    seq_of(a, b, start, L);
    const int64_t base = a.sq[b], square = (int64_t)L * L;
    if (base < 0 || base + square > a.total_square) continue;
    const int64_t e0 = (item - items[b]) * R_FLAT;              // < 2^32
    const int left = (int)(square - e0 < R_FLAT ? square - e0 : R_FLAT);
    const int i0 = (int)((uint32_t)e0 / (uint32_t)L), j0 = (int)(e0 - (int64_t)i0 * L);
    const float rl = 1.0f / (float)L;
    // row and column of this lane's elements, then what of them every head
    // shares: bucket (8 bits) and position index (17 bits), log2(1 + |dt|)
    uint32_t key[R_FSTEP];
    float l2[R_FSTEP];
#pragma unroll
    for (int k = 0; k < R_FSTEP; ++k) {
      const int x = j0 + 64 * k + lane;                         // < L + 1024 < 2^17
      int q = (int)((float)x * rl);                             // x / L, off by one at most
      int j = x - q * L;
      if (j < 0) { j += L; --q; }
      if (j >= L) { j -= L; ++q; }
      int i = i0 + q;
      i = i < L ? i : L - 1;                                    // past the square: not stored
      key[k] = (uint32_t)(j - i + a.N - 1) << 8;
      if (TIME || FN) {
        const int64_t dt = a.ts[start + i] - a.ts[start + j];
        if (TIME) key[k] |= (uint32_t)time_bucket32(dt, a.nb);
        if (FN) l2[k] = fn_lg2(dt);
      }
    }
    float *out = a.rab + base + e0;
    for (int h = 0; h < a.H; ++h) {
      const float *tab = TIME ? ttab + h * a.nb : nullptr;
      const float *pw = POS ? a.pos_w + h * span : nullptr;
      const float fa = FN ? a.time_fn[2 * h] : 0.0f, fb = FN ? a.time_fn[2 * h + 1] : 0.0f;
      float v[R_FSTEP];
#pragma unroll
      for (int k = 0; k < R_FSTEP; ++k) v[k] = POS ? pw[key[k] >> 8] : 0.0f;
#pragma unroll
      for (int k = 0; k < R_FSTEP; ++k) {
        if (TIME) v[k] += tab[key[k] & 255u];
        if (FN) v[k] += fa * __builtin_amdgcn_exp2f(-fb * l2[k]);
      }
      if (left == R_FLAT) {
#pragma unroll
        for (int k = 0; k < R_FSTEP; ++k) out[64 * k + lane] = v[k];
      } else {
#pragma unroll
        for (int k = 0; k < R_FSTEP; ++k)
          if (64 * k + lane < left) out[64 * k + lane] = v[k];
      }
      out += a.total_square;
    }
  }
}

// Sum of a double over the wave (the same order every time).
__device__ __forceinline__ double wave_sum_d(double x) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) x += __shfl_xor(x, m, 64);
  return x;
}

// Work-group of heads h0 .. h0 + HB - 1.  Dynamic LDS: their time histograms,
// [HB][nb][copies] (if time_w).
template <bool POS, bool TIME, bool FN, int HB>
__global__ void __launch_bounds__(R_BWD_THREADS, 4) rab_bwd_kernel(RabArgs a) {
  constexpr int WAVES = R_BWD_THREADS / 64;
  __shared__ int64_t s_items[R_LDS_SEQS + 1];
  __shared__ double red[2 * HB][WAVES];
  __shared__ int32_t s_cols[WAVES][64 + R_ROWS];
  extern __shared__ unsigned long long hist[];
  const int tid = threadIdx.x, lane = tid & 63;
  if (TIME)
    for (int x = tid; x < HB * a.nb * a.copies; x += R_BWD_THREADS) hist[x] = 0;
  const int64_t *items = stage_items(a, s_items, tid, R_BWD_THREADS);
  __syncthreads();
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int groups = a.H / HB;
  const int h0 = blockIdx.x % groups * HB, wg = blockIdx.x / groups, nwg = gridDim.x / groups;
  const int64_t n_items = items[a.B], span = 2 * (int64_t)a.N - 1;
  unsigned long long *mine = hist + (lane & (a.copies - 1));
  int32_t *cols = s_cols[w];
  float fb[HB];
  double s_a[HB], s_b[HB];              // sums of d g and d g log2(1 + |dt|)
  double run[HB];                       // this lane's run of bucket `cur`
#pragma unroll
  for (int u = 0; u < HB; ++u) {
    fb[u] = FN ? a.time_fn[2 * (h0 + u) + 1] : 0.0f;
    s_a[u] = s_b[u] = run[u] = 0.0;
  }
  int cur = 0;
  auto flush = [&]() {
#pragma unroll
    for (int u = 0; u < HB; ++u) {
      if (run[u] != 0.0) atomicAdd(&mine[(u * a.nb + cur) * a.copies], fix_d(run[u]));
      run[u] = 0.0;
    }
  };
  for (int64_t item = (int64_t)wg * WAVES + w; item < n_items; item += (int64_t)nwg * WAVES) {
    Strip t;
    if (!strip_of(a, items, item, t)) continue;
    const int d = t.d0 + lane;
    int32_t row = 0;
    bool near = true;
    if (TIME || FN) {
      const int64_t *ts = a.ts + t.start;
      const int64_t ts0 = ts[0];
      auto rel = [&](int x) {
        const int64_t r = ts[x < 0 ? 0 : (x < t.L ? x : t.L - 1)] - ts0;
        near &= r < R_NEAR && r > -R_NEAR;
        return (int32_t)r;
      };
      row = rel(t.r0 + (lane & (R_ROWS - 1)));
      const int c0 = t.r0 + t.d0;
      cols[lane] = rel(c0 + lane);
      if (lane < R_ROWS) cols[64 + lane] = rel(c0 + 64 + lane);
      near = __all(near);
      wave_lds_fence();
    }
    double diag[HB];
#pragma unroll
    for (int u = 0; u < HB; ++u) diag[u] = 0.0;
    for (int k0 = 0; k0 < t.rows; k0 += R_STEP) {
      const uint32_t ok = step_ok(t, k0, d);
      if (!__any(ok != 0)) continue;
      const float *in = a.d_rab + (int64_t)h0 * a.total_square + t.base +
                        (int64_t)(t.r0 + k0) * (t.L + 1) + t.d0;
      float g[HB][R_STEP];
      const bool full = __all(ok == (1u << R_STEP) - 1u);
#pragma unroll
      for (int u = 0; u < HB; ++u) {
        if (full) {
#pragma unroll
          for (int k = 0; k < R_STEP; ++k) g[u][k] = in[(uint32_t)(k * (t.L + 1) + lane)];
        } else {
#pragma unroll
          for (int k = 0; k < R_STEP; ++k)
            g[u][k] = (ok >> k) & 1 ? in[(uint32_t)(k * (t.L + 1) + lane)] : 0.0f;
        }
        in += a.total_square;
      }
      int bk[R_STEP];
      float l2[R_STEP];
      if (TIME || FN) step_keys<TIME, FN>(a, t, k0, lane, near, cols, row, bk, l2);
#pragma unroll
      for (int k = 0; k < R_STEP; ++k) {
        if (TIME && ((ok >> k) & 1) && bk[k] != cur) {
          flush();
          cur = bk[k];
        }
#pragma unroll
        for (int u = 0; u < HB; ++u) {
          const double gd = (double)g[u][k];
          if (POS) diag[u] += gd;
          if (TIME) run[u] += gd;
          if (FN) {
            const double ge = (double)(g[u][k] * __builtin_amdgcn_exp2f(-fb[u] * l2[k]));
            s_a[u] += ge;
            s_b[u] = __builtin_fma(ge, (double)l2[k], s_b[u]);
          }
        }
      }
    }
    if (POS) {
#pragma unroll
      for (int u = 0; u < HB; ++u)
        if (diag[u] != 0.0)
          atomicAdd(&a.fix_pos[(int64_t)(h0 + u) * span + d + a.N - 1], fix_d(diag[u]));
    }
    wave_lds_fence();
  }
  if (TIME) flush();
  if (FN) {
#pragma unroll
    for (int u = 0; u < HB; ++u) {
      const double x = wave_sum_d(s_a[u]), y = wave_sum_d(s_b[u]);
      if (lane == 0) { red[2 * u][w] = x; red[2 * u + 1][w] = y; }
    }
  }
  __syncthreads();
  if (FN && tid < 2 * HB) {
    double s = 0.0;
    for (int x = 0; x < WAVES; ++x) s += red[tid][x];
    // d of the exponent: -a ln(1 + |dt|) = -a ln 2 log2(1 + |dt|)
    if (tid & 1) s *= -(double)a.time_fn[2 * h0 + tid - 1] * TABLE_UNIT;
    if (s != 0.0) atomicAdd(&a.fix_fn[2 * h0 + tid], fix_d(s));
  }
  if (TIME) {
    for (int x = tid; x < HB * a.nb; x += R_BWD_THREADS) {
      unsigned long long s = 0;
      for (int c = 0; c < a.copies; ++c) s += hist[x * a.copies + ((c + x) & (a.copies - 1))];
      if (s != 0) atomicAdd(&a.fix_time[(int64_t)h0 * a.nb + x], s);
    }
  }
}

// The table sums as float, each table into its own output.
__global__ void rab_tables_out_kernel(RabArgs a, float *d_pos, float *d_time, float *d_fn) {
  const int64_t n_pos = d_pos ? (int64_t)a.H * (2 * (int64_t)a.N - 1) : 0;
  const int64_t n_time = d_time ? (int64_t)a.H * a.nb : 0, n_fn = d_fn ? 2 * (int64_t)a.H : 0;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n_pos + n_time + n_fn;
       x += (int64_t)gridDim.x * blockDim.x) {
    const int64_t y = x - n_pos, z = y - n_time;
    const unsigned long long *src = x < n_pos ? a.fix_pos + x : y < n_time ? a.fix_time + y
                                                                           : a.fix_fn + z;
    float *dst = x < n_pos ? d_pos + x : y < n_time ? d_time + y : d_fn + z;
    *dst = (float)((double)(long long)*src * (1.0 / FIX_ONE));
  }
}

// ------------------------------------------------------------------- host
int check_rab(const int64_t *off, int32_t B, int32_t N, int32_t H, int64_t T,
              int64_t total_square, const hstu_rab_params *rp) {
  if (B < 0) return fail(HSTU_EINVAL, "B = %d < 0", B);
  if (N < 1 || N > 65536) return fail(HSTU_EINVAL, "max_len = %d outside [1, 65536]", N);
  if (H < 1 || H > 64) return fail(HSTU_EINVAL, "H = %d outside [1, 64]", H);
  if (T < 0 || total_square < 0)
    return fail(HSTU_EINVAL, "total_tokens and total_square must be >= 0");
  if (!off && B > 0) return fail(HSTU_EINVAL, "seq_offsets must be non-null");
  if (!rp) return fail(HSTU_EINVAL, "rp is NULL");
  if ((rp->time_w || rp->time_fn) && !rp->timestamps && T > 0)
    return fail(HSTU_EINVAL, "time_w or time_fn given without timestamps");
  if (rp->time_w && (rp->num_buckets < 1 || (int64_t)H * rp->num_buckets > 4096))
    return fail(HSTU_EINVAL, "num_buckets = %d (need >= 1 and H * num_buckets <= 4096)",
                rp->num_buckets);
  return HSTU_OK;
}

struct RabLayout {
  size_t sq, items, fpos, ftime, ffn, total;
};

RabLayout rab_layout(int32_t B, int32_t N, int32_t H, const hstu_rab_params *rp) {
  RabLayout L{};
  size_t o = 0;
  auto take = [&](size_t bytes) { const size_t at = o; o = align_up(o + bytes); return at; };
  L.sq = take(sizeof(int64_t) * ((size_t)B + 1));
  L.items = take(sizeof(int64_t) * ((size_t)B + 1));
  L.fpos = rp->pos_w ? take(8 * (size_t)H * (2 * (size_t)N - 1)) : 0;
  L.ftime = rp->time_w ? take(8 * (size_t)H * rp->num_buckets) : 0;
  L.ffn = rp->time_fn ? take(8 * 2 * (size_t)H) : 0;
  L.total = o;
  return L;
}

RabArgs rab_args(const int64_t *off, int32_t B, int32_t N, int32_t H, int64_t T,
                 int64_t total_square, const hstu_rab_params *rp, char *ws,
                 const RabLayout &L) {
  RabArgs a{};
  a.off = off;
  a.sq = (int64_t *)(ws + L.sq);
  a.items = (int64_t *)(ws + L.items);
  a.pos_w = rp->pos_w;
  a.time_w = rp->time_w;
  a.time_fn = rp->time_fn;
  a.ts = (rp->time_w || rp->time_fn) ? rp->timestamps : nullptr;
  a.fix_pos = rp->pos_w ? (unsigned long long *)(ws + L.fpos) : nullptr;
  a.fix_time = rp->time_w ? (unsigned long long *)(ws + L.ftime) : nullptr;
  a.fix_fn = rp->time_fn ? (unsigned long long *)(ws + L.ffn) : nullptr;
  // the sums' regions follow each other (gaps and all) up to the layout's end
  const size_t first = rp->pos_w ? L.fpos : rp->time_w ? L.ftime : rp->time_fn ? L.ffn : L.total;
  a.fix = (unsigned long long *)(ws + first);
  a.n_fix = (int64_t)((L.total - first) / 8);
  a.T = T;
  a.total_square = total_square;
  a.B = B;
  a.N = N;
  a.H = H;
  a.nb = rp->time_w ? rp->num_buckets : 0;
  return a;
}

int rab_cus() {
  int dev = 0;
  (void)hipGetDevice(&dev);
  return device_info(dev).num_cu;
}

// Work-groups of `waves` waves for a batch: `per_cu` on every compute unit,
// fewer where the batch has fewer items (about one per 1024 elements of a
// head, and at least one per sequence).
int rab_grid(const RabArgs &a, int waves, int per_cu) {
  const int64_t items = a.total_square / 1024 + 2 * (int64_t)a.B;
  return (int)std::max<int64_t>(
      1, std::min<int64_t>((int64_t)per_cu * rab_cus(), (items + waves - 1) / waves));
}

template <int HB>
void launch_rab_bwd_t(RabArgs a, const hstu_rab_params *rp, hipStream_t s) {
  const bool P = rp->pos_w, Tm = rp->time_w, F = rp->time_fn;
  auto kfn = P ? (Tm ? (F ? rab_bwd_kernel<true, true, true, HB>
                          : rab_bwd_kernel<true, true, false, HB>)
                     : (F ? rab_bwd_kernel<true, false, true, HB>
                          : rab_bwd_kernel<true, false, false, HB>))
               : (Tm ? (F ? rab_bwd_kernel<false, true, true, HB>
                          : rab_bwd_kernel<false, true, false, HB>)
                     : (F ? rab_bwd_kernel<false, false, true, HB>
                          : rab_bwd_kernel<false, false, false, HB>));
  a.copies = 64;
  while ((int64_t)a.copies * a.nb * HB > R_HIST) a.copies >>= 1;
  const size_t dyn = rp->time_w ? 8 * (size_t)a.copies * a.nb * HB : 0;
  const int groups = a.H / HB;
  const int per_group = std::min(rab_grid(a, R_BWD_THREADS / 64, 2),
                                 std::max(1, 2 * rab_cus() / groups));
  hipLaunchKernelGGL(kfn, dim3((unsigned)(groups * per_group)), dim3(R_BWD_THREADS), dyn, s, a);
}

void launch_rab_bwd(const RabArgs &a, const hstu_rab_params *rp, hipStream_t s) {
  if (a.H % 2 == 0) launch_rab_bwd_t<2>(a, rp, s);
  else launch_rab_bwd_t<1>(a, rp, s);
}

}  // namespace
}  // namespace hstu

using namespace hstu;

extern "C" size_t hstu_jagged_rab_workspace_bytes(int32_t B, int32_t max_len, int32_t H,
                                                  const hstu_rab_params *rp) {
  clear_last_error();
  static const int64_t dummy = 0;
  if (check_rab(&dummy, B, max_len, H, 0, 0, rp)) return 0;
  return rab_layout(B, max_len, H, rp).total;
}

extern "C" int hstu_jagged_rab_fwd(const int64_t *seq_offsets, int32_t B, int32_t max_len,
                                   int32_t H, int64_t total_tokens, int64_t total_square,
                                   const hstu_rab_params *rp, float *rab, void *workspace,
                                   size_t workspace_bytes, void *stream) {
  clear_last_error();
  int rc = check_rab(seq_offsets, B, max_len, H, total_tokens, total_square, rp);
  if (rc) return rc;
  if (B == 0 || total_square == 0) return HSTU_OK;
  if (!rab) return fail(HSTU_EINVAL, "rab must be non-null");
  const RabLayout L = rab_layout(B, max_len, H, rp);
  if ((rc = check_workspace_bytes(L.total, workspace, workspace_bytes))) return rc;
  const hipStream_t s = (hipStream_t)stream;
  RabArgs a = rab_args(seq_offsets, B, max_len, H, total_tokens, total_square, rp,
                       (char *)workspace, L);
  a.rab = rab;
  prof::Scope ps("rab_fwd", s);
  hipLaunchKernelGGL(rab_scan_kernel, dim3(1), dim3(R_SCAN_THREADS), 0, s, a);
  const bool P = rp->pos_w, Tm = rp->time_w, F = rp->time_fn;
  auto kfn = P ? (Tm ? (F ? rab_fwd_kernel<true, true, true> : rab_fwd_kernel<true, true, false>)
                     : (F ? rab_fwd_kernel<true, false, true> : rab_fwd_kernel<true, false, false>))
               : (Tm ? (F ? rab_fwd_kernel<false, true, true> : rab_fwd_kernel<false, true, false>)
                     : (F ? rab_fwd_kernel<false, false, true>
                          : rab_fwd_kernel<false, false, false>));
  hipLaunchKernelGGL(kfn, dim3((rab_grid(a, R_FWD_THREADS / 64, 8) + 7) / 8 * 8), dim3(R_FWD_THREADS),
                     rp->time_w ? sizeof(float) * (size_t)H * rp->num_buckets : 0, s, a);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? HSTU_OK : hip_fail(e, "rab forward launch");
}

extern "C" int hstu_jagged_rab_bwd(const int64_t *seq_offsets, int32_t B, int32_t max_len,
                                   int32_t H, int64_t total_tokens, int64_t total_square,
                                   const hstu_rab_params *rp, const float *d_rab,
                                   float *d_pos_w, float *d_time_w, float *d_time_fn,
                                   void *workspace, size_t workspace_bytes, void *stream) {
  clear_last_error();
  int rc = check_rab(seq_offsets, B, max_len, H, total_tokens, total_square, rp);
  if (rc) return rc;
  if ((rp->pos_w && !d_pos_w) || (rp->time_w && !d_time_w) || (rp->time_fn && !d_time_fn))
    return fail(HSTU_EINVAL, "a gradient output is NULL for a given parameter");
  if (B > 0 && total_square > 0 && !d_rab) return fail(HSTU_EINVAL, "d_rab must be non-null");
  const RabLayout L = rab_layout(B, max_len, H, rp);
  if ((rc = check_workspace_bytes(L.total, workspace, workspace_bytes))) return rc;
  const hipStream_t s = (hipStream_t)stream;
  char *ws = (char *)workspace;
  RabArgs a = rab_args(seq_offsets, B, max_len, H, total_tokens, total_square, rp, ws, L);
  a.d_rab = d_rab;
  const int64_t n_pos = (int64_t)H * (2 * (int64_t)max_len - 1);
  const int64_t n_time = rp->time_w ? (int64_t)H * rp->num_buckets : 0;
  prof::Scope ps("rab_bwd", s);
  const bool any = B > 0 && total_square > 0;
  if (!any) a.B = 0;
  const int64_t zero_blocks = std::min<int64_t>(256, (a.n_fix + R_SCAN_THREADS - 1) / R_SCAN_THREADS);
  hipLaunchKernelGGL(rab_scan_kernel, dim3((unsigned)(1 + zero_blocks)), dim3(R_SCAN_THREADS), 0,
                     s, a);
  if (any) {
    launch_rab_bwd(a, rp, s);
  }
  const int64_t n_out = (d_pos_w && a.fix_pos ? n_pos : 0) + n_time + (a.fix_fn ? 2 * H : 0);
  if (n_out > 0)
    hipLaunchKernelGGL(rab_tables_out_kernel,
                       dim3((unsigned)std::min<int64_t>(256, (n_out + 255) / 256)), dim3(256), 0,
                       s, a, a.fix_pos ? d_pos_w : nullptr, a.fix_time ? d_time_w : nullptr,
                       a.fix_fn ? d_time_fn : nullptr);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? HSTU_OK : hip_fail(e, "rab backward launch");
}
