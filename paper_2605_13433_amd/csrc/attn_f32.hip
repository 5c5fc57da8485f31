// float32 jagged HSTU attention (forward and backward) on the fp32 matrix
// cores of gfx950.
//
// Same definition as the bf16 kernels with every operand, product and sum in
// fp32 (v_mfma_f32_32x32x2_f32; the two bias-table gradients are summed in
// float64 or 64-bit fixed point).
//
// An item is a 32-row half of one 64-row work-list tile of one head: 32
// queries for the forward and dQ, 32 keys for dK/dV.  The four waves (NW; two
// for batches of many short sequences, two_waves) of a work-group take every
// fourth 32-row tile of the item's streamed side, each on its own -- a wave
// stages its tile in its own part of the LDS, so the loop has no barrier; each
// operand's loads are in flight under the product before it, through one set of
// registers -- and their partial sums are added through LDS in wave order at the
// end (the result does not depend on timing).
//
// What bounds it: a 32 x 32 tile is D/2 matrix instructions of 64 cycles for
// every product, and a batch of short sequences is as long as its longest
// item.  Hence 32-row items split over four waves (a 512-token sequence's
// longest dK/dV item is 4 tiles deep in every wave), and the score-side
// products read their streamed operand by rows out of LDS (16 bytes a lane)
// while the accumulating products use the scores where the first product
// left them: its accumulator register r holds streamed row c_row(r, g) of
// this lane's stationary row, which is the B operand of a K = 2 step over
// rows c_row(r, 0) and c_row(r, 1).
// Measured against one thread per row on the vector ALUs (48 power-law
// sequences of 16..512 tokens, H = 4, d = 64, both biases): forward 582 ->
// 30 us, backward 7796 -> 108 us (6886 of them were one double atomic on a
// table entry per pair); four sequences of up to 64 tokens, H = 2, d = 32:
// forward 27 -> 6.5 us.  Error against 64 bits (relative, the whole output), nine
// batches of 37 to 432 sequences, d = 32, 64 and 128, two draws each: o 0.64 to
// 0.94 times the former kernels', dv 0.66 to 0.96, y and du 0.75 to 1.02, dq and
// dk 0.7 to 1.2 (a few short sequences' LayerNorm decides those); on the batch
// above o 3.0e-7 -> 2.1e-7, dk 4.2e-7 -> 3.6e-7.
// What is left beside the chain of tiles: the d = 64 backward spills registers
// (the 256-register cap), and every score gathers its two biases from memory.
// Matrix cores busy 16% of the cycles, the vector ALUs 13%.
#include <algorithm>

#include "internal.h"
#include "device.h"
#include "attn_common.h"
#include "sched_impl.h"

namespace hstu {

namespace {

constexpr int FT = 32;                     // rows of an item and of a streamed tile
// A work-group's d_time histogram sits in LDS (hist_copies_log2 counters a
// bucket) up to this many buckets; above it every finished run goes straight
// to the table.
constexpr int F32_LDS_BUCKETS = 512;

struct F32Params {
  const float *q, *k, *v, *dO;
  const float *pos_w, *time_w;
  const int64_t *ts;
  const int32_t *ctrl;
  const WorkEntry *list_q, *list_k;
  float *o, *dq, *dk, *dv;
  // table-gradient sums in the workspace: double (default mode; many
  // thousands of terms land on one entry, more than float keeps to 1e-5 of
  // the table) or 64-bit fixed point (deterministic mode)
  void *acc_pos, *acc_time;
  int32_t H, N, nb;
  float inv_n, alpha;
  // direct forward: no lists, each work-group's item found from the offsets
  const int64_t *off;
  int64_t T;
  int32_t B, direct, max_entries;
  int32_t time_cs;                // log2 of the histogram's counters per bucket
};

// K = 2 step of a 32 x 32 product: lane l gives A[l % 32][l / 32] and
// B[l / 32][l % 32]; the accumulator has the layout of mfma32's.
__device__ __forceinline__ f32x16 mfma2(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// The thread index as a value the compiler cannot trace back: per-lane
// addresses are rebuilt for each item instead of living across them.
__device__ __forceinline__ int opaque_tid() {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  return tid;
}

template <int D> constexpr int F32_ROW = D + 4;       // LDS row: the 16 rows of a 16-byte
                                                      // read phase fall on all 64 banks

// The rows of one head of a sequence as a buffer source: rows at or past the
// sequence's length read as zeros.  At most 65536 * 64 * 128 * 4 = 2^31 bytes.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_of(const F32Params &P, const float *p,
                                                          const WorkEntry &e, int h, int D) {
  const uint32_t row = 4u * (uint32_t)(P.H * D);
  // up to the end of the last row's D floats, not of the whole last row
  return make_rsrc(p + (e.start * P.H + h) * D, (uint32_t)(e.len - 1) * row + 4u * (uint32_t)D);
}

// Stationary rows of an item, one per lane: lane (l32, g) holds dims g D/2 ..
// of row row0 + l32.
template <int D>
__device__ __forceinline__ void load_rows(const F32Params &P, __amdgpu_buffer_rsrc_t rs, int row,
                                          int g, float (&reg)[D / 2]) {
  const uint32_t at = 4u * (uint32_t)(P.H * D) * (uint32_t)row + 2u * (uint32_t)(g * D);
#pragma unroll
  for (int x = 0; x < D / 8; ++x) {
    const float4 f = __builtin_bit_cast(float4, buf_load16(rs, at + 16u * x));
    reg[4 * x] = f.x; reg[4 * x + 1] = f.y; reg[4 * x + 2] = f.z; reg[4 * x + 3] = f.w;
  }
}

// A 32-row tile of one head on its way to LDS, 16-byte chunks of a wave.
template <int D>
struct F32Tile {
  static constexpr int CH = FT * D / 4 / 64;
  uint4 c[CH];
  static constexpr int RPC = 64 / (D / 4);          // rows per chunk step
  __device__ __forceinline__ void load(const F32Params &P, __amdgpu_buffer_rsrc_t rs, int row0,
                                       int lane) {
    const uint32_t row_bytes = 4u * (uint32_t)(P.H * D);
    const uint32_t at = row_bytes * (uint32_t)(row0 + lane / (D / 4)) + 16u * (lane % (D / 4));
#pragma unroll
    for (int x = 0; x < CH; ++x) c[x] = buf_load16(rs, at + (uint32_t)(x * RPC) * row_bytes);
  }
  __device__ __forceinline__ void store(float *lds, int lane) const {
#pragma unroll
    for (int x = 0; x < CH; ++x) {
      const int ch = lane + 64 * x, row = ch / (D / 4), col = ch % (D / 4);
      *(uint4 *)(lds + row * F32_ROW<D> + 4 * col) = c[x];
    }
  }
};

// Product of the tile's rows in LDS (rows of the result) with the
// stationary rows (columns): result register r of lane (l32, g) is tile row
// c_row(r, g) times stationary row l32.
template <int D>
__device__ __forceinline__ f32x16 tile_scores(const float *lds, const float (&st)[D / 2], int l32,
                                              int g) {
  f32x16 s;
#pragma unroll
  for (int r = 0; r < 16; ++r) s[r] = 0.0f;
  const float *p = lds + l32 * F32_ROW<D> + g * (D / 2);
#pragma unroll
  for (int x = 0; x < D / 8; ++x) {
    const float4 f = *(const float4 *)(p + 4 * x);
    s = mfma2(f.x, st[4 * x], s);
    s = mfma2(f.y, st[4 * x + 1], s);
    s = mfma2(f.z, st[4 * x + 2], s);
    s = mfma2(f.w, st[4 * x + 3], s);
  }
  return s;
}

// acc[db] += X^T P: X = the tile's rows in LDS, P the pair values in the
// layout tile_scores leaves them in.  acc register r of lane (l32, g) is dim
// 32 db + c_row(r, g) of stationary row l32.  On an `edge` tile some pairs do
// not exist (their value is 0; `ok` bit r: pair (c_row(r, g), l32) does):
// should X hold an infinity or NaN, which 0 would not cancel, those elements
// are added for the existing pairs alone and leave the tile first.
template <int D>
__device__ __forceinline__ void tile_accumulate(float *lds, const float (&p)[16], bool edge,
                                                uint32_t ok, int l32, int g,
                                                f32x16 (&acc)[D / 32]) {
  if (edge) {
    bool bad = false;
#pragma unroll 4
    for (int x = l32 + 32 * g; x < FT * D; x += 64)
      bad |= !(__builtin_fabsf(lds[(x / D) * F32_ROW<D> + x % D]) < __builtin_inff());
    if (__any(bad)) {
      auto odd = [](float f) { return !(__builtin_fabsf(f) < __builtin_inff()); };
#pragma unroll 1
      for (int row = 0; row < FT; ++row) {
        const int src = l32 + 32 * ((row >> 2) & 1), reg = 4 * (row >> 3) + (row & 3);
        float pv = 0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r) pv = r == reg ? p[r] : pv;
        pv = __shfl(pv, src, 64);
        const bool have = (__shfl((int)ok, src, 64) >> reg) & 1;
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float f = lds[row * F32_ROW<D> + 32 * db + c_row(r, g)];
            if (have && odd(f)) acc[db][r] = __builtin_fmaf(pv, f, acc[db][r]);
          }
      }
      wave_lds_fence();
      for (int x = l32 + 32 * g; x < FT * D; x += 64) {
        float &f = lds[(x / D) * F32_ROW<D> + x % D];
        if (odd(f)) f = 0.0f;
      }
      wave_lds_fence();
    }
  }
#pragma unroll
  for (int r = 0; r < 16; ++r)
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
      acc[db] = mfma2(lds[c_row(r, g) * F32_ROW<D> + 32 * db + l32], p[r], acc[db]);
}

// Sum of the NW waves' accumulators (each through its own LDS part, in
// wave order) and the store of the item's rows (those below `valid`) times
// `scale`.  With `more`, on top of what an earlier call stored with scale 1
// (every thread reads back its own elements).
template <int D, int NW>
__device__ __forceinline__ void sum_store(float *lds0, int part, const f32x16 (&acc)[D / 32],
                                          int tid, float *out, int row_stride, int valid,
                                          float scale, bool more = false) {
  const int lane = tid & 63, l32 = lane & 31, g = lane >> 5;
  float *mine = lds0 + (tid >> 6) * part;
  __syncthreads();
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *(float4 *)(mine + l32 * F32_ROW<D> + 32 * db + 8 * q + 4 * g) =
          make_float4(acc[db][4 * q], acc[db][4 * q + 1], acc[db][4 * q + 2], acc[db][4 * q + 3]);
  __syncthreads();
#pragma unroll
  for (int x = 0; x < FT * D / 4 / (64 * NW); ++x) {
    const int ch = tid + 64 * NW * x, row = ch / (D / 4), col = ch % (D / 4);
    if (row >= valid) continue;
    float *dst = out + (int64_t)row * row_stride + 4 * col;
    float4 s = *(const float4 *)(lds0 + row * F32_ROW<D> + 4 * col);
    if (NW == 2 && more) {
      const float4 b = *(const float4 *)dst;
      s.x += b.x; s.y += b.y; s.z += b.z; s.w += b.w;
    }
#pragma unroll
    for (int w = 1; w < NW; ++w) {
      const float4 t = *(const float4 *)(lds0 + w * part + row * F32_ROW<D> + 4 * col);
      s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
    }
    *(float4 *)dst = make_float4(scale * s.x, scale * s.y, scale * s.z, scale * s.w);
  }
}

template <int D>
__device__ __forceinline__ void clear(f32x16 (&acc)[D / 32]) {
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[db][r] = 0.0f;
}

// The bias sources of one head of one item.
struct F32Bias {
  __amdgpu_buffer_rsrc_t pos;          // the head's position table (0 outside it)
  const float *time;
  int64_t ts_own;                      // timestamp of this lane's stationary row
};

__device__ __forceinline__ F32Bias bias_of(const F32Params &P, const WorkEntry &e, int h,
                                           int row) {
  F32Bias b;
  const int span = 2 * P.N - 1;
  b.pos = make_rsrc(P.pos_w ? P.pos_w + (int64_t)h * span : P.q,
                    P.pos_w ? 4u * (uint32_t)span : 0u);
  b.time = P.time_w ? P.time_w + (int64_t)h * P.nb : nullptr;
  b.ts_own = P.time_w ? P.ts[e.start + (row < e.len ? row : e.len - 1)] : 0;
  return b;
}

// Time buckets of a lane's 16 pairs, four to a register (a bucket is at most
// 4 * 62 + 3).
struct Buckets {
  uint32_t b[4];
  __device__ __forceinline__ int at(int r) const { return (int)((b[r >> 2] >> (8 * (r & 3))) & 255u); }
};

// s = alpha s + (position + time bias) of the tile's pairs: the biases are added
// first, so that two that cancel leave the score its precision.  `off` = j - i
// of the pair of streamed row 0 and this lane's stationary row, `dir` the change
// of j - i per streamed row (+1 where the streamed side is keys, -1 queries);
// `bk` receives the time buckets.  The scheduling barrier keeps the bias loads
// out of the products' registers.
__device__ __forceinline__ void add_bias(const F32Params &P, const F32Bias &b, f32x16 &s, int off,
                                         int dir, const int64_t *ts, int g, Buckets &bk) {
  __builtin_amdgcn_sched_barrier(0);
  float w[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) w[r] = 0.0f;
  if (P.pos_w) {
#pragma unroll
    for (int r = 0; r < 16; ++r) w[r] = pos_entry(b.pos, off + dir * c_row(r, g) + P.N - 1);
  }
  if (P.time_w) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      bk.b[q] = 0;
#pragma unroll
      for (int c = 0; c < 4; ++c)
        bk.b[q] |= (uint32_t)time_bucket32(b.ts_own - ts[c_row(4 * q + c, g)], P.nb) << (8 * c);
      __builtin_amdgcn_sched_barrier(0);
    }
    float tw[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) tw[r] = b.time[bk.at(r)];
#pragma unroll
    for (int r = 0; r < 16; ++r) w[r] += tw[r];
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) s[r] = __builtin_fmaf(P.alpha, s[r], w[r]);
}

// Timestamps of the streamed tile in the wave's part of LDS (rows past the
// sequence repeat its last one; their pairs do not exist).
__device__ __forceinline__ void stage_ts(const F32Params &P, const WorkEntry &e, int row0,
                                         int64_t *ts, int lane) {
  if (P.time_w && lane < FT) {
    const int r = row0 + lane;
    ts[lane] = P.ts[e.start + (r < e.len ? r : e.len - 1)];
  }
}

// Pairs of a tile whose streamed rows are keys row0.. and this lane's query
// i, or (KEYS false) queries row0.. and this lane's key: bit r set where the
// pair exists.
template <bool KEYS>
__device__ __forceinline__ uint32_t pair_bits(int row0, int own, int len, int g) {
  uint32_t ok = 0;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int x = row0 + c_row(r, g);
    const bool have = KEYS ? x <= own && own < len : x >= own && x < len;
    ok |= have ? 1u << r : 0u;
  }
  return ok;
}

// Work item `item` of `list`: entry, head and 32-row half; false if the half
// lies past the sequence.
__device__ __forceinline__ bool item_of(const F32Params &P, const WorkEntry *list, int64_t item,
                                        WorkEntry &e, int &h, int &row0) {
  const int64_t eh = item >> 1;
  const int64_t entry = eh / P.H;
  h = (int)(eh - entry * P.H);
  if (P.direct) {
    if (!direct_entry(P.off, P.B, P.N, P.T, (int)entry, e)) return false;
  } else {
    e = list[entry];
  }
  row0 = e.tile * TILE + FT * (int)(item & 1);
  return row0 < e.len;
}

// Whether an item of `tiles` streamed tiles goes into its second round after
// this wave's tile (two waves only, see two_waves: at most four tiles, so both
// waves meet here).  The first round's sum is then stored and the waves start
// anew, so that every sum is the one of four waves with a tile each, added in
// the same order: a sequence has the same bits in either form.
template <int NW>
__device__ __forceinline__ bool second_round(int tile, int tiles) {
  return NW == 2 && tile < NW && tiles > NW;
}

template <int D, int NW>
struct F32FwdSmem {
  float tile[NW][2][FT * F32_ROW<D>];     // K, V of each wave's tile
  int64_t ts[NW][FT];
};

template <int D, int NW>
__device__ __forceinline__ void f32_fwd_item(const F32Params &P, F32FwdSmem<D, NW> &sm,
                                             int64_t item) {
  WorkEntry e;
  int h, i0;
  if (!item_of(P, P.list_q, item, e, h, i0)) return;
  const int tid = opaque_tid(), lane = tid & 63, l32 = lane & 31, g = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = i0 + l32;
  float *ks = sm.tile[w][0], *vs = sm.tile[w][1];
  const __amdgpu_buffer_rsrc_t rq = rows_of(P, P.q, e, h, D), rk = rows_of(P, P.k, e, h, D),
                               rv = rows_of(P, P.v, e, h, D);
  F32Tile<D> t;
  t.load(P, rk, FT * w, lane);
  float qreg[D / 2];
  load_rows<D>(P, rq, i, g, qreg);
  const F32Bias bias = bias_of(P, e, h, i);
  f32x16 acc[D / 32];
  clear<D>(acc);
  float *out = P.o + ((e.start + i0) * P.H + h) * D;

  const int last = i0 / FT;
  for (int kt = w; kt <= last; kt += NW) {
    const int j0 = FT * kt;
    t.store(ks, lane);
    stage_ts(P, e, j0, sm.ts[w], lane);
    wave_lds_fence();
    t.load(P, rv, j0, lane);
    f32x16 s = tile_scores<D>(ks, qreg, l32, g);
    t.store(vs, lane);
    wave_lds_fence();
    t.load(P, rk, j0 + FT * NW, lane);
    Buckets bk;
    add_bias(P, bias, s, j0 - i, 1, sm.ts[w], g, bk);
    const bool edge = kt == last;
    float a[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) a[r] = s[r] * sigmoid_f(s[r]) * P.inv_n;
    uint32_t ok = 0;
    if (edge) {
      ok = pair_bits<true>(j0, i, e.len, g);
#pragma unroll
      for (int r = 0; r < 16; ++r) a[r] = (ok >> r) & 1 ? a[r] : 0.0f;
    }
    tile_accumulate<D>(vs, a, edge, ok, l32, g, acc);
    wave_lds_fence();
    if (second_round<NW>(kt, last + 1)) {
      sum_store<D, NW>(&sm.tile[0][0][0], 2 * FT * F32_ROW<D>, acc, tid, out, P.H * D, e.len - i0,
                       1.0f);
      clear<D>(acc);
      __syncthreads();                  // the next tile overwrites what was read
    }
  }
  sum_store<D, NW>(&sm.tile[0][0][0], 2 * FT * F32_ROW<D>, acc, tid, out, P.H * D, e.len - i0,
                   1.0f, last >= NW);
}

template <int D, int NW>
__global__ void __launch_bounds__(64 * NW, D == 128 ? 1 : 2)
f32_fwd_kernel(F32Params P) {
  __shared__ __attribute__((aligned(16))) F32FwdSmem<D, NW> sm;
  if (P.direct && blockIdx.x == 0 && threadIdx.x == 0)
    const_cast<int32_t *>(P.ctrl)[CTRL_STATUS] = HSTU_SEQ_UNCHECKED;
  const int64_t n_items = 2 * (int64_t)(P.direct ? P.max_entries : P.ctrl[CTRL_N_ENTRIES]) * P.H;
  for (int64_t item = blockIdx.x; item < n_items; item += gridDim.x) {
    f32_fwd_item<D, NW>(P, sm, item);
    __syncthreads();
  }
}

// Table-gradient sums: LDS and global in double, or (deterministic mode)
// 64-bit fixed point, whose integer additions give the same result in any
// order.
template <bool DET> struct F32Tab;
template <> struct F32Tab<false> {
  typedef double T;
  static __device__ __forceinline__ T of(float v) { return (double)v; }
};
template <> struct F32Tab<true> {
  typedef unsigned long long T;
  static __device__ __forceinline__ T of(float v) { return to_fix(v); }
};

template <int D, bool DET, int NW>
struct F32BwdSmem {
  float tile[NW][2][FT * F32_ROW<D>];     // K, V or Q, dO of each wave's tile
  int64_t ts[NW][FT];
  // diagonal sums of each wave's tile, one copy per lane group (the lanes of
  // an atomic hit distinct slots)
  typename F32Tab<DET>::T win[NW][2][2 * FT];
};

template <int D, bool DET, int NW>
__device__ __forceinline__ void f32_dq_item(const F32Params &P, F32BwdSmem<D, DET, NW> &sm,
                                            int64_t item) {
  WorkEntry e;
  int h, i0;
  if (!item_of(P, P.list_q, item, e, h, i0)) return;
  const int tid = opaque_tid(), lane = tid & 63, l32 = lane & 31, g = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = i0 + l32;
  float *ks = sm.tile[w][0], *vs = sm.tile[w][1];
  const __amdgpu_buffer_rsrc_t rk = rows_of(P, P.k, e, h, D), rv = rows_of(P, P.v, e, h, D);
  F32Tile<D> t;
  t.load(P, rk, FT * w, lane);
  float qreg[D / 2], oreg[D / 2];
  load_rows<D>(P, rows_of(P, P.q, e, h, D), i, g, qreg);
  load_rows<D>(P, rows_of(P, P.dO, e, h, D), i, g, oreg);
  const F32Bias bias = bias_of(P, e, h, i);
  f32x16 acc[D / 32];
  clear<D>(acc);
  float *out = P.dq + ((e.start + i0) * P.H + h) * D;

  const int last = i0 / FT;
  for (int kt = w; kt <= last; kt += NW) {
    const int j0 = FT * kt;
    t.store(ks, lane);
    stage_ts(P, e, j0, sm.ts[w], lane);
    wave_lds_fence();
    t.load(P, rv, j0, lane);
    f32x16 s = tile_scores<D>(ks, qreg, l32, g);
    t.store(vs, lane);
    wave_lds_fence();
    t.load(P, rk, j0 + FT * NW, lane);
    const f32x16 da = tile_scores<D>(vs, oreg, l32, g);
    Buckets bk;
    add_bias(P, bias, s, j0 - i, 1, sm.ts[w], g, bk);
    const bool edge = kt == last;
    float ds[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float sg = sigmoid_f(s[r]);
      ds[r] = da[r] * sg * (1.0f + s[r] * (1.0f - sg)) * P.inv_n;
    }
    uint32_t ok = 0;
    if (edge) {
      ok = pair_bits<true>(j0, i, e.len, g);
#pragma unroll
      for (int r = 0; r < 16; ++r) ds[r] = (ok >> r) & 1 ? ds[r] : 0.0f;
    }
    tile_accumulate<D>(ks, ds, edge, ok, l32, g, acc);
    wave_lds_fence();
    if (second_round<NW>(kt, last + 1)) {
      sum_store<D, NW>(&sm.tile[0][0][0], 2 * FT * F32_ROW<D>, acc, tid, out, P.H * D, e.len - i0,
                       1.0f);
      clear<D>(acc);
      __syncthreads();                  // the next tile overwrites what was read
    }
  }
  sum_store<D, NW>(&sm.tile[0][0][0], 2 * FT * F32_ROW<D>, acc, tid, out, P.H * D, e.len - i0,
                   P.alpha, last >= NW);
}

template <int D, bool DET, int NW>
__device__ __forceinline__ void f32_dkv_item(const F32Params &P, F32BwdSmem<D, DET, NW> &sm,
                                             typename F32Tab<DET>::T *hist, int64_t item) {
  typedef F32Tab<DET> A;
  WorkEntry e;
  int h, j0;
  if (!item_of(P, P.list_k, item, e, h, j0)) return;
  const int tid = opaque_tid(), lane = tid & 63, l32 = lane & 31, g = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = j0 + l32;
  const int first = j0 / FT, tiles = (e.len + FT - 1) / FT;
  float *qs = sm.tile[w][0], *os = sm.tile[w][1];
  const __amdgpu_buffer_rsrc_t rq = rows_of(P, P.q, e, h, D), ro = rows_of(P, P.dO, e, h, D);
  F32Tile<D> t;
  t.load(P, rq, j0 + FT * w, lane);
  float kreg[D / 2], vreg[D / 2];
  load_rows<D>(P, rows_of(P, P.k, e, h, D), j, g, kreg);
  load_rows<D>(P, rows_of(P, P.v, e, h, D), j, g, vreg);
  const F32Bias bias = bias_of(P, e, h, j);
  const bool time_g = P.acc_time != nullptr;
  const bool in_lds = P.nb <= F32_LDS_BUCKETS;
  typename A::T *gt = time_g ? (typename A::T *)P.acc_time + (int64_t)h * P.nb : nullptr;
  typename A::T *gp = P.acc_pos
                          ? (typename A::T *)P.acc_pos + (int64_t)h * (2 * (int64_t)P.N - 1)
                          : nullptr;
  for (int x = lane; x < 4 * FT; x += 64) (&sm.win[w][0][0])[x] = 0;
  if (time_g && in_lds)
    for (int x = tid; x < P.nb << P.time_cs; x += 64 * NW) hist[x] = 0;
  // runs of equal buckets down this lane's queries, also from tile to tile
  // (ordered timestamps change bucket rarely), summed like the table
  typename A::T run = 0;
  int cur = -1;
  auto flush = [&]() {
    if (in_lds) atomicAdd(&hist[(cur << P.time_cs) + (lane & ((1 << P.time_cs) - 1))], run);
    else atomicAdd(&gt[cur], run);
  };
  __syncthreads();
  f32x16 dk[D / 32], dv[D / 32];
  clear<D>(dk);
  clear<D>(dv);
  const int64_t at = ((e.start + j0) * P.H + h) * D;

  for (int qt = first + w; qt < tiles; qt += NW) {
    const int i0 = FT * qt;
    t.store(qs, lane);
    stage_ts(P, e, i0, sm.ts[w], lane);
    wave_lds_fence();
    t.load(P, ro, i0, lane);
    f32x16 s = tile_scores<D>(qs, kreg, l32, g);
    t.store(os, lane);
    wave_lds_fence();
    t.load(P, rq, i0 + FT * NW, lane);
    const f32x16 da = tile_scores<D>(os, vreg, l32, g);
    Buckets bk;
    add_bias(P, bias, s, j - i0, -1, sm.ts[w], g, bk);
    const bool edge = qt == first || qt == tiles - 1 || j0 + FT > e.len;
    float a[16], ds[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float sg = sigmoid_f(s[r]);
      a[r] = s[r] * sg * P.inv_n;
      ds[r] = da[r] * sg * (1.0f + s[r] * (1.0f - sg)) * P.inv_n;
    }
    uint32_t ok = 0xffffu;
    if (edge) {
      ok = pair_bits<false>(i0, j, e.len, g);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        a[r] = (ok >> r) & 1 ? a[r] : 0.0f;
        ds[r] = (ok >> r) & 1 ? ds[r] : 0.0f;
      }
    }
    if (gp) {
      // slot i - j + 31 (- the tile's offset) of this lane group's window,
      // then the window's 63 diagonals to the table
      typename A::T *pw = &sm.win[w][g][FT - 1 - l32];
#pragma unroll
      for (int r = 0; r < 16; ++r) atomicAdd(pw + c_row(r, g), A::of(ds[r]));
      wave_lds_fence();
      const typename A::T v = sm.win[w][0][lane] + sm.win[w][1][lane];
      sm.win[w][0][lane] = 0;
      sm.win[w][1][lane] = 0;
      const int m = i0 - j0 + lane - (FT - 1);
      if (v != 0 && m >= 0 && m < e.len) atomicAdd(&gp[P.N - 1 - m], v);
    }
    if (time_g) {
      cur = cur < 0 ? bk.at(0) : cur;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if (bk.at(r) != cur) {
          flush();
          run = 0;
          cur = bk.at(r);
        }
        run += A::of(ds[r]);
      }
    }
    tile_accumulate<D>(os, a, edge, ok, l32, g, dv);
    tile_accumulate<D>(qs, ds, edge, ok, l32, g, dk);
    wave_lds_fence();
    if (second_round<NW>(qt - first, tiles - first)) {
      sum_store<D, NW>(&sm.tile[0][0][0], 2 * FT * F32_ROW<D>, dk, tid, P.dk + at, P.H * D,
                       e.len - j0, 1.0f);
      sum_store<D, NW>(&sm.tile[0][0][0], 2 * FT * F32_ROW<D>, dv, tid, P.dv + at, P.H * D,
                       e.len - j0, 1.0f);
      clear<D>(dk);
      clear<D>(dv);
      __syncthreads();                  // the next tile overwrites what was read
    }
  }
  if (time_g && cur >= 0) flush();
  sum_store<D, NW>(&sm.tile[0][0][0], 2 * FT * F32_ROW<D>, dk, tid, P.dk + at, P.H * D,
                   e.len - j0, P.alpha, tiles - first > NW);
  sum_store<D, NW>(&sm.tile[0][0][0], 2 * FT * F32_ROW<D>, dv, tid, P.dv + at, P.H * D,
                   e.len - j0, 1.0f, tiles - first > NW);
  if (time_g && in_lds)
    for (int x = tid; x < P.nb; x += 64 * NW) {
      typename A::T v = 0;
      for (int c = 0; c < 1 << P.time_cs; ++c) v += hist[(x << P.time_cs) + c];
      if (v != 0) atomicAdd(&gt[x], v);
    }
}

// Both item kinds of the backward in one launch, a dK/dV and a dQ item in
// turn down the longest-first lists, so that neither kind's tail is alone.
template <int D, bool DET, int NW>
__global__ void __launch_bounds__(64 * NW, D == 128 ? 1 : 2)
f32_bwd_kernel(F32Params P) {
  __shared__ __attribute__((aligned(16))) F32BwdSmem<D, DET, NW> sm;
  extern __shared__ double dyn_f32[];              // d_time histogram of the item's head
  const int64_t n_items = 4 * (int64_t)P.ctrl[CTRL_N_ENTRIES] * P.H;
  for (int64_t item = blockIdx.x; item < n_items; item += gridDim.x) {
    if (item & 1) f32_dq_item<D, DET, NW>(P, sm, item >> 1);
    else f32_dkv_item<D, DET, NW>(P, sm, (typename F32Tab<DET>::T *)dyn_f32, item >> 1);
    __syncthreads();
  }
}

// The two tables' sums cleared, and converted to float (either may be absent).
__global__ void f32_tables_zero_kernel(unsigned long long *pos, int64_t n_pos,
                                       unsigned long long *time, int64_t n_time) {
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n_pos + n_time;
       x += (int64_t)gridDim.x * blockDim.x)
    (x < n_pos ? pos[x] : time[x - n_pos]) = 0;
}

template <bool DET>
__global__ void f32_tables_out_kernel(const void *pos, int64_t n_pos, const void *time,
                                      int64_t n_time, float *d_pos, float *d_time) {
  typedef typename F32Tab<DET>::T T;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n_pos + n_time;
       x += (int64_t)gridDim.x * blockDim.x) {
    const bool p = x < n_pos;
    const T v = p ? ((const T *)pos)[x] : ((const T *)time)[x - n_pos];
    const float f = DET ? (float)((double)(long long)v * (1.0 / FIX_ONE)) : (float)v;
    if (p) d_pos[x] = f;
    else d_time[x - n_pos] = f;
  }
}

// One work-group per item (`per` of them to a list entry and head) up to a
// million, which then take the rest in turn.
dim3 f32_grid(const Problem &p, int per) {
  return dim3((unsigned)std::max<int64_t>(
      1, std::min<int64_t>((int64_t)1 << 20, per * p.max_entries * p.H)));
}

// Two waves a work-group instead of four where sequences have at most four
// 32-row tiles and the work-groups (`per` to a list entry and head) queue for
// the device: the third and fourth wave of most items would have no tile, and
// only hold their place.  Forward / backward (us), four waves and two: 300
// sequences of up to 100 tokens, 8 heads of 64, 141 / 518 and 102 / 438; 200 of
// up to 110, 8 heads of 128, 257 / 900 and 182 / 672; 300 of up to 128, 4 heads of
// 32, 51 / 190 and 48 / 135; just above the line, 48 of 100..128, 4 heads of 64,
// 31 / 82 and 30 / 82; but 4 of 60..128, 2 heads of 64, 12 / 25 and 15 / 34, where
// the chain of tiles doubles.  (Without second_round, whose sums spill: 96 / 414,
// 168 / 561, 41 / 127, 28 / 74, and other bits than four waves give.)  Resident to
// a compute unit with four waves: one at d = 128, three of the d = 32 forward (48 of
// 100..128, 4 heads, which all fit: 20.0 with four and 21.2 with two), else two.
bool two_waves(const Problem &p, int per) {
  int dev = 0;
  (void)hipGetDevice(&dev);
  const int resident = p.d == 128 ? 1 : p.d == 32 && per == 2 ? 3 : 2;
  return p.N <= 4 * FT && per * p.max_entries * p.H > resident * (int64_t)device_info(dev).num_cu;
}

template <int NW>
auto pick_fwd(int d) {
  return d == 32 ? f32_fwd_kernel<32, NW> : d == 64 ? f32_fwd_kernel<64, NW>
                                                    : f32_fwd_kernel<128, NW>;
}
template <bool DET, int NW>
auto pick_bwd(int d) {
  return d == 32 ? f32_bwd_kernel<32, DET, NW> : d == 64 ? f32_bwd_kernel<64, DET, NW>
                                                         : f32_bwd_kernel<128, DET, NW>;
}

F32Params make_params(const AttnArgs &a) {
  const char *ws = (const char *)a.ws;
  F32Params P{};
  P.q = (const float *)a.q;
  P.k = (const float *)a.k;
  P.v = (const float *)a.v;
  P.pos_w = a.pos_w;
  P.time_w = a.time_w;
  P.ts = a.ts;
  P.ctrl = (const int32_t *)(ws + a.L.ctrl);
  P.list_q = (const WorkEntry *)(ws + a.L.list_q);
  P.list_k = (const WorkEntry *)(ws + a.L.list_k);
  P.H = a.p.H;
  P.N = a.p.N;
  P.nb = a.p.has_time ? a.p.nb : 0;
  P.inv_n = 1.0f / (float)a.p.N;
  P.alpha = a.p.alpha;
  return P;
}

}  // namespace

hipError_t launch_attn_fwd_f32(const AttnArgs &a, void *o, bool direct, hipStream_t s) {
  F32Params P = make_params(a);
  if (direct) {
    P.off = a.off;
    P.T = a.p.T;
    P.B = a.p.B;
    P.max_entries = (int32_t)a.p.max_entries;
    P.direct = 1;
  }
  P.o = (float *)o;
  const bool two = two_waves(a.p, 2);
  auto kfn = two ? pick_fwd<2>(a.p.d) : pick_fwd<4>(a.p.d);
  hipLaunchKernelGGL(kfn, f32_grid(a.p, 2), dim3(two ? 128 : 256), 0, s, P);
  return hipGetLastError();
}

hipError_t launch_attn_bwd_f32(const AttnArgs &a, const void *dO, void *dq,
                               void *dk, void *dv, float *d_pos, float *d_time,
                               hipStream_t s) {
  const char *ws = (const char *)a.ws;
  const Problem &p = a.p;
  // table-shaped sums in the workspace (8 bytes per entry): 64-bit fixed
  // point in the deterministic mode, double otherwise; converted to the
  // float tables after the kernel (zeros when T = 0)
  const int64_t n_pos = d_pos ? (int64_t)p.H * (2 * (int64_t)p.N - 1) : 0;
  const int64_t n_time = d_time ? (int64_t)p.H * p.nb : 0;
  void *st_pos = d_pos ? (void *)(ws + a.L.dpos_part) : nullptr;
  void *st_time = d_time ? (void *)(ws + a.L.dtime_part) : nullptr;
  const bool tables = n_pos + n_time > 0;
  const dim3 tgrid((unsigned)std::min<int64_t>(256, (n_pos + n_time + 255) / 256));
  hipError_t e = hipSuccess;
  if (tables) {
    hipLaunchKernelGGL(f32_tables_zero_kernel, tgrid, dim3(256), 0, s,
                       (unsigned long long *)st_pos, n_pos, (unsigned long long *)st_time, n_time);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (p.T > 0) {
    F32Params P = make_params(a);
    P.dO = (const float *)dO;
    P.dq = (float *)dq;
    P.dk = (float *)dk;
    P.dv = (float *)dv;
    P.acc_pos = st_pos;
    P.acc_time = st_time;
    P.time_cs = hist_copies_log2(p.nb);
    const size_t dyn =
        d_time && p.nb <= F32_LDS_BUCKETS ? sizeof(double) * (size_t)p.nb << P.time_cs : 0;
    const bool two = two_waves(p, 4);
    auto kfn = p.deterministic ? (two ? pick_bwd<true, 2>(p.d) : pick_bwd<true, 4>(p.d))
                               : (two ? pick_bwd<false, 2>(p.d) : pick_bwd<false, 4>(p.d));
    hipLaunchKernelGGL(kfn, f32_grid(p, 4), dim3(two ? 128 : 256), dyn, s, P);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (tables) {
    auto kfn = p.deterministic ? f32_tables_out_kernel<true> : f32_tables_out_kernel<false>;
    hipLaunchKernelGGL(kfn, tgrid, dim3(256), 0, s, (const void *)st_pos, n_pos,
                       (const void *)st_time, n_time, d_pos, d_time);
  }
  return hipGetLastError();
}

}  // namespace hstu
