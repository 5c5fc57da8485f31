// Pieces shared by the bf16 attention kernels of gfx950: the base-2 score
// domain, the float-exponent time index and its runs, the LDS transpose read
// and the table-gradient accumulation types.
#pragma once

#include "internal.h"
#include "device.h"

namespace hstu {

constexpr int KTAB = 608;        // float-exponent time index 0..603 (+pad)
constexpr int32_t NEAR = 1 << 23;  // |ts - ts_start| < NEAR -> float-exponent path
constexpr float L2E = 1.44269504088896341f;      // log2(e)

typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16;

// Float-exponent index of a time difference held exactly in a float
// (|delta| < 2^24; see file comment).  The sign bit is not in the field.
__device__ __forceinline__ int time_index(float delta) {
  return (int)__builtin_amdgcn_ubfe(__float_as_uint(delta), 21u, 10u);
}

// Bucket of float-exponent index k (k = 0 <-> 0; 508, 512, 514 <-> 1, 2, 3;
// k >= 516 <-> k - 512), clamped to nb-1.  Indices no integer reaches map
// to some valid bucket.
__device__ __forceinline__ int bucket_of_index(int k, int nb) {
  int b = k >= 516 ? k - 512 : (k >= 514 ? 3 : (k >= 512 ? 2 : (k >= 508 ? 1 : 0)));
  return b < nb - 1 ? b : nb - 1;
}

// Scores are handled in the base-2 domain x' = x log2(e): the MFMA result is
// scaled once and the bias tables are staged pre-scaled, so that e^-x is a
// single exp2 of -x'.
//   silu(x) / N = x' / (N log2e (1 + 2^-x'));  nl = N log2e
__device__ __forceinline__ float silu2_over_n(float xs, float nl) {
  const float t = __builtin_amdgcn_exp2f(-xs);
  return xs * __builtin_amdgcn_rcpf(__builtin_fmaf(nl, t, nl));
}

// The forward's score of a pair in that domain, s alpha log2(e) + time bias'.
// Rounded once (`xs` not used) at d = 64 with a position bias and twice
// elsewhere (xs = scaled_score(s, al2e)), by name: the compiler fuses the product
// into the sum in one instantiation and not in the next, and a sequence's bits
// must not depend on which kernel its batch took.
template <int D, bool POS> constexpr bool TIME_FUSED = D == 64 && POS;
__device__ __forceinline__ float scaled_score(float s, float al2e) {
#pragma clang fp contract(off)
  const float x = s * al2e;
  return x;
}
template <int D, bool POS>
__device__ __forceinline__ float time_score(float s, float xs, float al2e, float tb) {
  return TIME_FUSED<D, POS> ? __builtin_fmaf(s, al2e, tb) : xs + tb;
}

// Entry `idx` of a position table that is a buffer source: 0 outside the table,
// one dword by itself.  The index is opaque because the compiler merges loads of
// neighbouring entries, and a wide load whose first word lies before the table
// reads 0 in all of them: the items whose streamed rows are queries walk the
// table downwards, past its beginning in the last rows of a sequence of max_len.
__device__ __forceinline__ float pos_entry(__amdgpu_buffer_rsrc_t rs, int idx) {
  asm("" : "+v"(idx));
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, 4 * idx, 0, 0));
}

// Operand holding, for lane l, column ncol + (l & 31) of rows krow .. krow+3
// and krow+8 .. krow+11 of a row-major LDS tile (krow already includes this
// lane's 4*(l/32)), via two LDS transpose loads.  Within a 16-lane group,
// lane c addresses row (c>>2), columns 4*(c&3)..+3 of its group's 16-column
// slab; the transpose hands lane i the column slab+i of the four rows.
__device__ __forceinline__ bf16x8 read_tr(const u16 *lds, int stride, int krow,
                                          int ncol, int lane) {
  const int c = lane & 15;
  const u16 *p = lds + (krow + (c >> 2)) * stride + ncol + ((lane >> 4) & 1) * 16 + 4 * (c & 3);
  const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16 *)p);
  const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16 *)(p + 8 * stride));
  typedef short v8i16 __attribute__((ext_vector_type(8)));
  const v8i16 x = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, x);
}

// The backward's dS of a pair from sg = sigma(score) and da = <dO, v>, in natural
// units for dQ.  The score is alpha x (biases staged divided by alpha):
// silu'(alpha x) = sigma (1 + x (alpha - alpha sigma)).
__device__ __forceinline__ float dq_ds(float sg, float da, float x, float alpha) {
  return (sg * da) * __builtin_fmaf(x, __builtin_fmaf(-alpha, sg, alpha), 1.0f);
}

// As dq_ds for dK/dV, which carry a = silu and dS = dA silu' = dA (sg + a (1 - sg))
// multiplied by log2e (A' = u sg with u = score log2e, dS' = dA (sg log2e +
// A' (1 - sg))): one multiply per element fewer than natural units; the stores
// divide it out, and the table partials keep it until the finalize pass.
__device__ __forceinline__ float dkv_ds(float a, float sg, float da) {
  return da * __builtin_fmaf(-a, sg, __builtin_fmaf(sg, L2E, a));
}

// Table-gradient accumulation types: LDS sums in double and global partials
// in float (d_pos: one per sequence and diagonal) or double (d_time: one per
// item), or (deterministic mode) all as 64-bit fixed point, whose integer
// additions give the same result in any order.
template <bool DET> struct TabAcc {
  typedef double L;
  typedef float G;
  typedef double GT;
  static __device__ __forceinline__ L lds(float v) { return (double)v; }
  static __device__ __forceinline__ G glob(L v) { return (float)v; }
};
template <> struct TabAcc<true> {
  typedef unsigned long long L;
  typedef unsigned long long G;
  typedef unsigned long long GT;
  static __device__ __forceinline__ L lds(float v) { return to_fix(v); }
  static __device__ __forceinline__ G glob(L v) { return v; }
};

// Per-lane running sum of d_time contributions (dS multiplied by log2e, as
// the dK/dV items carry it; the table partials keep that factor, which the
// finalize pass divides out) over one float-exponent time index (the lane's
// pairs visit non-decreasing indices when timestamps are ordered, so a run
// ends only when its index changes); a finished run goes to its bucket of
// the item's histogram `hist` (2^cs counters a bucket, see hist_copies).  A run is
// opened by
// the first index of the item's first tile (start), so adding needs no test
// for an empty run.
template <typename A>
struct TimeRun {
  typedef typename A::L L;
  float sum = 0.0f;
  int cur = -1;
  __device__ __forceinline__ void start(int k) { cur = cur < 0 ? k : cur; }
  __device__ __forceinline__ void add(L *hist, int nb, int cs, int k, float v) {
    const bool change = k != cur;
    if (change) atomicAdd(&hist[bucket_of_index(cur, nb) << cs], A::lds(sum));
    sum = change ? v : sum + v;
    cur = k;
  }
  __device__ __forceinline__ void flush(L *hist, int nb, int cs) {
    if (cur >= 0) atomicAdd(&hist[bucket_of_index(cur, nb) << cs], A::lds(sum));
    cur = -1;
    sum = 0.0f;
  }
};

// log2 of the counters per bucket of an item's d_time histogram: lanes are
// spread over them, because neighbouring keys meet in the same bucket and a
// wave's LDS atomics on one address are served one by one (44 clocks for four
// lanes, 8 for none).  Up to eight, in at most `bytes`.
constexpr int64_t HIST_BYTES = 4096;
inline int hist_copies_log2(int nb, int64_t bytes = HIST_BYTES) {
  int cs = 3;
  while (cs > 0 && ((int64_t)nb << cs) * 8 > bytes) --cs;
  return cs;
}

}  // namespace hstu
