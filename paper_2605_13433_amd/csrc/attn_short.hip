// bf16 MFMA attention for batches that leave the tile kernels of
// attn_bf16.hip idle: short sequences, or few of them.
//
// There a work-group walks a 64-row item's partner tiles one after another,
// two barriers or one a step, so a call is as long as its longest item's
// chain of steps, and a short item is mostly its start and its end.  Here an
// item is 32 rows of one head and its four waves take every fourth 32-row
// tile of the other side:
//
//   * a wave loads its tile's rows from memory straight into the layout of the
//     score products (lane: one row, 16 bytes at a time), on its own;
//   * the chain is a quarter as long in tiles of half the rows.
//
// A step's four tiles and their packed scores meet in the LDS, and the
// accumulating products are dealt out by what they add to, so that every sum is
// added up in the tile kernels' order and a sequence has the same bits whichever
// kernel its batch takes.  Forward, dQ, and dK/dV at d = 64: each wave has the
// even or the odd tiles (the halves of the tile kernels' 64 rows) and half of the
// dims; dK/dV at d = 128: one of the two and half of the dims, over every tile.
// dQ has room for two buffers and needs one barrier a step; the others have two,
// the forward's one after the other with only the stores between them.
// Summed by each wave for itself and added at the end, without a barrier, the
// forward for one sequence of 502 / 812 / 2 heads of 8022 tokens took 11.8 / 15.2 /
// 103 us and takes 11.7 / 15.4 / 110 (d = 128, 502: 17.6 and 16.2), the backward
// of 8 sequences of up to 100 tokens at d = 128 20.8 and 19.2, of one of 502 / 812
// 27.4 / 37.1 and 27.7 / 38.7, of one of 2000 at d = 128 72 and 85: the waves wait
// for the slowest one's table sums in every step.
// Forward with two buffers and one barrier: 11.2 / 14.9 / 107, but 54 KB, which
// leaves a compute unit two work-groups instead of three.
//
// Per score the work is that of the tile kernels (same operands, same
// roundings, the base-2 domain), and every 32 rows stream the other side
// once instead of every 64 (or 128): the kernels cost more traffic and lose
// where the device is full (fwd_short and bwd_short have the line and what
// both sides measured).
#include <algorithm>

#include "internal.h"
#include "device.h"
#include "attn_common.h"
#include "sched_impl.h"

namespace hstu {

namespace {

constexpr int S_THREADS = 256;               // 4 waves
constexpr int S_WAVES = S_THREADS / 64;
constexpr int ST = 32;                       // rows of an item and of a streamed tile
template <int D> constexpr int S_ROW = D + 8;    // LDS row of a tile (bf16)
template <int D> constexpr int S_RED = D + 4;    // LDS row of a partial sum (float)

struct SParams {
  const u16 *q, *k, *v, *dO;
  const float *pos_w, *time_w;
  const int64_t *ts, *off;
  int32_t *ctrl;
  const WorkEntry *list_q, *list_k;
  u16 *o, *dq, *dk, *dv;
  const u16 *h_dq, *h_dk, *h_dv;             // silu' factors of the gradients (or null)
  int32_t out_stride;                        // row stride of the gradients (elements)
  void *dpos_part, *dtime_part;              // see TabAcc
  int64_t T;
  int32_t B, H, N, nb, direct;
  int32_t time_cs;                           // log2 of the d_time counters per bucket
  float alpha, inv_alpha, neg_al2e, al2e, dqk_scale, dk_scale_l2, dv_scale_l2;
};

// Item `item` of the batch: list entry, head and 32-row half.  False past
// the last entry or the sequence.
__device__ __forceinline__ bool short_item(const SParams &P, const WorkEntry *list, int item,
                                           WorkEntry &e, int &h, int &row0) {
  const int eh = item >> 1, entry = eh / P.H;
  h = eh - entry * P.H;
  if (P.direct) {
    if (!direct_entry(P.off, P.B, P.N, P.T, entry, e)) return false;
  } else {
    if (entry >= P.ctrl[CTRL_N_ENTRIES]) return false;
    e = list[entry];
  }
  row0 = e.tile * TILE + ST * (item & 1);
  return row0 < e.len;
}

// The rows of one head of a sequence: rows at or past its length read 0.
template <int D>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t head_rows(const SParams &P, const u16 *p,
                                                            const WorkEntry &e, int h) {
  const uint32_t row = 2u * (uint32_t)(P.H * D);
  return make_rsrc(p + (e.start * P.H + h) * D, (uint32_t)(e.len - 1) * row + 2u * (uint32_t)D);
}

// 32 rows in the layout of the score products: lane (l32, g) holds dims
// 16 ks + 8 g .. + 7 of row row0 + l32.
template <int D>
struct Rows {
  uint4 r[D / 16];
  __device__ __forceinline__ void load(const SParams &P, __amdgpu_buffer_rsrc_t rs, int row,
                                       int g) {
    const uint32_t at = 2u * (uint32_t)(P.H * D) * (uint32_t)row + 16u * (uint32_t)g;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) r[ks] = buf_load16(rs, at + 32u * ks);
  }
  __device__ __forceinline__ void store(u16 *lds, int l32, int g) const {
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks)
      *(uint4 *)(lds + l32 * S_ROW<D> + 16 * ks + 8 * g) = r[ks];
  }
};

// s += X Y^T: result register r of lane (l32, g) is row c_row(r, g) of X
// times row l32 of Y.
template <int D>
__device__ __forceinline__ f32x16 score(const Rows<D> &x, const Rows<D> &y, f32x16 s) {
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) s = mfma32(as_bf16x8(x.r[ks]), as_bf16x8(y.r[ks]), s);
  return s;
}

__device__ __forceinline__ uint4 pack8(const float (&f)[8]) {
  return make_uint4(pack2(f[0], f[1]), pack2(f[2], f[3]), pack2(f[4], f[5]), pack2(f[6], f[7]));
}

// Position table of a head as a buffer source (entries outside it read 0).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t pos_table(const SParams &P, bool on, int h) {
  const int span = 2 * P.N - 1;
  return make_rsrc(on ? P.pos_w + (int64_t)h * span : (const float *)P.q,
                   on ? 4u * (uint32_t)span : 0u);
}

// Position biases of this lane's 16 pairs, offset j - i = off + DIR c_row(r, 0).
// Up the table the compiler may merge four entries into one load: existing rows
// begin inside it.
template <int DIR>
__device__ __forceinline__ void load_pos(const SParams &P, __amdgpu_buffer_rsrc_t rs, int off,
                                         float (&p)[16]) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int idx = off + DIR * c_row(r, 0) + P.N - 1;
    p[r] = DIR > 0 ? __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, 4 * idx, 0, 0))
                   : pos_entry(rs, idx);
  }
}

// Time side of an item: the head's table by float-exponent index in LDS
// (staged by the work-group, see attn_bf16.hip for the index), each wave's tile
// timestamps relative to the sequence's first.
struct ShortTime {
  float tab[KTAB];
  alignas(16) float rel[S_WAVES][ST];
};

__device__ __forceinline__ void stage_table(const SParams &P, ShortTime &t, int h, int tid,
                                            float scale) {
  const float *tw = P.time_w + (int64_t)h * P.nb;
#pragma unroll
  for (int x = 0; x < (KTAB + S_THREADS - 1) / S_THREADS; ++x) {
    const int i = tid + S_THREADS * x;
    if (i < KTAB) t.tab[i] = scale * tw[bucket_of_index(i, P.nb)];
  }
}

// The table's value for a gap outside the float-exponent index, scaled as
// stage_table scales it (rounded by itself: a product fused into the sum would
// differ from a staged one).
__device__ __forceinline__ float far_time(const SParams &P, int h, int64_t gap, float scale) {
#pragma clang fp contract(off)
  const float v = scale * P.time_w[(int64_t)h * P.nb + time_bucket(gap, P.nb)];
  return v;
}

// Timestamp of row `row` of the sequence (its last row's past the end).
__device__ __forceinline__ int64_t ts_of(const SParams &P, const WorkEntry &e, int row) {
  return P.ts[e.start + (row < e.len ? row : e.len - 1)];
}

// This lane's own row and the tile's rows on the time axis.  `slow`: some
// difference does not fit the float-exponent index; the exact rule on the
// timestamps runs instead.
struct TimeAxis {
  int64_t own, start;
  float own_rel;
  bool far;
  __device__ __forceinline__ void set(const SParams &P, const WorkEntry &e, int row) {
    start = P.ts[e.start];
    own = ts_of(P, e, row);
    const int64_t r = own - start;
    own_rel = (float)(int32_t)r;
    far = r >= NEAR || r <= -NEAR;
  }
  // Stages a tile's relative timestamps (lanes 0..31, `t` the lane's row's).
  __device__ __forceinline__ bool stage(float *rel, int64_t t, int lane) const {
    const int64_t r = t - start;
    if (lane < ST) rel[lane] = (float)(int32_t)r;
    return __any(far || (lane < ST && (r >= NEAR || r <= -NEAR)));
  }
};

// Packed scores of a step's four tiles, as the accumulating products take
// them: [tile][16-row half][lane].
typedef uint4 ShortPacks[S_WAVES][2][64];

// acc += X^T P over one streamed tile (its rows in LDS, its packed scores) for
// the NB 32-dim blocks from `db0` on.
template <int D, int NB>
__device__ __forceinline__ void accumulate_from(const u16 *lds, const uint4 (&p)[2][64], int db0,
                                                int g, int lane, f32x16 (&acc)[NB]) {
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    const bf16x8 b = as_bf16x8(p[hh][lane]);
#pragma unroll
    for (int y = 0; y < NB; ++y)
      acc[y] = mfma32(read_tr(lds, S_ROW<D>, 16 * hh + 4 * g, 32 * (db0 + y), lane), b, acc[y]);
  }
}

// An item's sums on their way out: a wave's NB blocks from dim 32 db0 on to a
// buffer of the item's rows, then (all waves, after a barrier) the rows below
// `valid` as bf16, times `scale` and, with `hsrc`, times silu' of the bf16 at
// the same place.  TWO: the sum of two buffers.
template <int D, int NB>
__device__ __forceinline__ void put_sums(float *buf, const f32x16 (&acc)[NB], int db0, int l32,
                                         int g) {
  float *p = buf + l32 * S_RED<D> + 32 * db0 + 4 * g;
#pragma unroll
  for (int y = 0; y < NB; ++y)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *(float4 *)(p + 32 * y + 8 * q) =
          make_float4(acc[y][4 * q], acc[y][4 * q + 1], acc[y][4 * q + 2], acc[y][4 * q + 3]);
}

template <int D, bool TWO>
__device__ __forceinline__ void emit_rows(const float *buf, int tid, u16 *out, int row_stride,
                                          int valid, float scale, const u16 *hsrc) {
#pragma unroll
  for (int x = 0; x < ST * D / 8 / S_THREADS; ++x) {
    const int ch = tid + S_THREADS * x, row = ch / (D / 8), c8 = ch % (D / 8);
    if (row >= valid) continue;
    float f[8];
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      float4 a = *(const float4 *)(buf + row * S_RED<D> + 8 * c8 + 4 * y);
      if constexpr (TWO) {
        const float4 b = *(const float4 *)(buf + (ST + row) * S_RED<D> + 8 * c8 + 4 * y);
        a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
      }
      f[4 * y] = scale * a.x;
      f[4 * y + 1] = scale * a.y;
      f[4 * y + 2] = scale * a.z;
      f[4 * y + 3] = scale * a.w;
    }
    const int64_t at = (int64_t)row * row_stride + 8 * c8;
    if (hsrc) {
      const uint4 hv = *(const uint4 *)(hsrc + at);
      const uint32_t hw[4] = {hv.x, hv.y, hv.z, hv.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        f[2 * e] *= dsilu_f(__uint_as_float(hw[e] << 16));
        f[2 * e + 1] *= dsilu_f(__uint_as_float(hw[e] & 0xffff0000u));
      }
    }
    *(uint4 *)(out + at) = pack8(f);
  }
}

template <int NB>
__device__ __forceinline__ void clear(f32x16 (&acc)[NB]) {
#pragma unroll
  for (int y = 0; y < NB; ++y)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[y][r] = 0.0f;
}

// ---------------------------------------------------------------- forward
template <int D>
struct ShortFwdSmem {
  union {
    struct {
      u16 v[S_WAVES][ST * S_ROW<D>];
      ShortPacks p;
    };
    float red[2][ST * S_RED<D>];
  };
  ShortTime t;
};

template <int D, bool POS, bool TIME>
__global__ void __launch_bounds__(S_THREADS, D == 64 ? 3 : 2) short_fwd_kernel(SParams P) {
  __shared__ __attribute__((aligned(16))) ShortFwdSmem<D> sm;
  if (P.direct && blockIdx.x == 0 && threadIdx.x == 0)
    P.ctrl[CTRL_STATUS] = HSTU_SEQ_UNCHECKED;
  WorkEntry e;
  int h, i0;
  if (!short_item(P, P.list_q, blockIdx.x, e, h, i0)) return;
  constexpr int NB = D / 64;                          // 32-dim blocks of a wave's half
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = i0 + l32, last = i0 / ST;
  const int par = w & 1, db0 = NB * (w >> 1);         // what this wave accumulates
  const __amdgpu_buffer_rsrc_t rk = head_rows<D>(P, P.k, e, h), rv = head_rows<D>(P, P.v, e, h),
                               rp = pos_table(P, POS, h);
  // everything the start needs is asked for at once
  Rows<D> kr, vr, qr;
  kr.load(P, rk, ST * w + l32, g);
  qr.load(P, head_rows<D>(P, P.q, e, h), i, g);
  vr.load(P, rv, ST * w + l32, g);
  float pw[16];
  if (POS) load_pos<1>(P, rp, ST * w + 4 * g - i, pw);
  TimeAxis ax{};
  int64_t tk = 0;
  if (TIME) {
    tk = ts_of(P, e, ST * w + l32);
    ax.set(P, e, i);
    stage_table(P, sm.t, h, tid, L2E);
    __syncthreads();
  }
  f32x16 acc[NB];
  clear(acc);
  const float nl = (float)P.N * L2E;

  for (int k0 = 0; k0 <= last; k0 += S_WAVES) {
    const int kt = k0 + w, j0 = ST * kt, nj = j0 + ST * S_WAVES;
    const bool have = kt <= last, more = kt + S_WAVES <= last;
    uint4 pk[2];
    if (have) {
      const bool slow = TIME && ax.stage(sm.t.rel[w], tk, lane);
      if (TIME) wave_lds_fence();
      f32x16 s;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = POS ? pw[r] * P.inv_alpha : 0.0f;
      s = score<D>(kr, qr, s);
      if (more) {                                     // the wave's next tile
        kr.load(P, rk, nj + l32, g);
        if (POS) load_pos<1>(P, rp, nj + 4 * g - i, pw);
        if (TIME) tk = ts_of(P, e, nj + l32);
      }
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        float x[8], a[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) x[c] = scaled_score(s[8 * hh + c], P.al2e);
        if (TIME) {
          if (!slow) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
              const float4 t4 = *(const float4 *)(sm.t.rel[w] + 16 * hh + 8 * q + 4 * g);
              const int r = 8 * hh + 4 * q;
              const float *tab = sm.t.tab;
              x[4 * q + 0] = time_score<D, POS>(s[r], x[4 * q + 0], P.al2e, tab[time_index(ax.own_rel - t4.x)]);
              x[4 * q + 1] = time_score<D, POS>(s[r + 1], x[4 * q + 1], P.al2e, tab[time_index(ax.own_rel - t4.y)]);
              x[4 * q + 2] = time_score<D, POS>(s[r + 2], x[4 * q + 2], P.al2e, tab[time_index(ax.own_rel - t4.z)]);
              x[4 * q + 3] = time_score<D, POS>(s[r + 3], x[4 * q + 3], P.al2e, tab[time_index(ax.own_rel - t4.w)]);
            }
          } else {
#pragma unroll
            for (int c = 0; c < 8; ++c)
              x[c] = time_score<D, POS>(
                  s[8 * hh + c], x[c], P.al2e,
                  far_time(P, h, ax.own - ts_of(P, e, j0 + c_row(8 * hh + c, g)), L2E));
          }
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) a[c] = silu2_over_n(x[c], nl);
        if (kt == last) {
#pragma unroll
          for (int c = 0; c < 8; ++c)
            if (j0 + c_row(8 * hh + c, g) > i) a[c] = 0.0f;
        }
        pk[hh] = pack8(a);
      }
    }
    if (k0 > 0) lds_barrier();                        // the step before is read
    if (have) {
      vr.store(sm.v[w], l32, g);
      sm.p[w][0][lane] = pk[0];
      sm.p[w][1][lane] = pk[1];
      if (more) vr.load(P, rv, nj + l32, g);
    }
    lds_barrier();
#pragma unroll
    for (int x = par; x < S_WAVES; x += 2)
      if (k0 + x <= last) accumulate_from<D>(sm.v[x], sm.p[x], db0, g, lane, acc);
  }
  lds_barrier();
  put_sums<D>(sm.red[par], acc, db0, l32, g);
  lds_barrier();
  emit_rows<D, true>(sm.red[0], tid, P.o + ((e.start + i0) * P.H + h) * D, P.H * D, e.len - i0,
                     1.0f, nullptr);
}

// --------------------------------------------------------------- backward
template <int D, bool DET>
struct ShortBwdSmem {
  union {
    struct {
      u16 x[S_WAVES][2][ST * S_ROW<D>];      // dQ: K, by the step's parity; dK/dV: Q, dO
      ShortPacks p[2];                       // dQ: by the step's parity; dK/dV: A, dS
    };
    float red[D == 64 ? 4 : 2][ST * S_RED<D>];
  };
  ShortTime t;
  // diagonal sums of each wave's tile, one copy per lane group
  typename TabAcc<DET>::L win[S_WAVES][2][2 * ST];
};

// At d = 64 the tile kernels' dK/dV items compute dQ of a sequence's first 64
// rows, out of their base-2 dS and in one chain over the keys; so do the items of
// those rows here.
template <int D, bool POS, bool TIME, bool DET>
__device__ __forceinline__ void short_dq(const SParams &P, ShortBwdSmem<D, DET> &sm, int item) {
  WorkEntry e;
  int h, i0;
  if (!short_item(P, P.list_q, item, e, h, i0)) return;
  constexpr int NB = D / 64;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = i0 + l32, last = i0 / ST;
  const int par = w & 1, db0 = NB * (w >> 1);
  const bool first64 = D == 64 && e.tile == 0;
  const __amdgpu_buffer_rsrc_t rk = head_rows<D>(P, P.k, e, h), rv = head_rows<D>(P, P.v, e, h),
                               rp = pos_table(P, POS, h);
  Rows<D> kr, vr, qr, dr;
  kr.load(P, rk, ST * w + l32, g);
  qr.load(P, head_rows<D>(P, P.q, e, h), i, g);
  vr.load(P, rv, ST * w + l32, g);
  dr.load(P, head_rows<D>(P, P.dO, e, h), i, g);
  float pw[16];
  if (POS) load_pos<1>(P, rp, ST * w + 4 * g - i, pw);
  TimeAxis ax{};
  int64_t tk = 0;
  if (TIME) {
    tk = ts_of(P, e, ST * w + l32);
    ax.set(P, e, i);
    stage_table(P, sm.t, h, tid, P.inv_alpha);
    __syncthreads();
  }
  f32x16 acc[NB];
  clear(acc);

  for (int k0 = 0, b = 0; k0 <= last; k0 += S_WAVES, b ^= 1) {
    const int kt = k0 + w, j0 = ST * kt, nj = j0 + ST * S_WAVES;
    if (kt <= last) {
      kr.store(sm.x[w][b], l32, g);
      const bool slow = TIME && ax.stage(sm.t.rel[w], tk, lane);
      if (TIME) wave_lds_fence();
      f32x16 s, da;
#pragma unroll
      for (int r = 0; r < 16; ++r) { s[r] = POS ? pw[r] * P.inv_alpha : 0.0f; da[r] = 0.0f; }
      s = score<D>(kr, qr, s);
      da = score<D>(vr, dr, da);
      if (kt + S_WAVES <= last) {
        kr.load(P, rk, nj + l32, g);
        vr.load(P, rv, nj + l32, g);
        if (POS) load_pos<1>(P, rp, nj + 4 * g - i, pw);
        if (TIME) tk = ts_of(P, e, nj + l32);
      }
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        float x[8], ds[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) x[c] = s[8 * hh + c];
        if (TIME) {
          if (!slow) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
              const float4 t4 = *(const float4 *)(sm.t.rel[w] + 16 * hh + 8 * q + 4 * g);
              x[4 * q + 0] += sm.t.tab[time_index(ax.own_rel - t4.x)];
              x[4 * q + 1] += sm.t.tab[time_index(ax.own_rel - t4.y)];
              x[4 * q + 2] += sm.t.tab[time_index(ax.own_rel - t4.z)];
              x[4 * q + 3] += sm.t.tab[time_index(ax.own_rel - t4.w)];
            }
          } else {
#pragma unroll
            for (int c = 0; c < 8; ++c)
              x[c] += far_time(P, h, ax.own - ts_of(P, e, j0 + c_row(8 * hh + c, g)), P.inv_alpha);
          }
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          if (first64) {
            const float u = x[c] * P.al2e;
            const float sg = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-u));
            ds[c] = dkv_ds(u * sg, sg, da[8 * hh + c]);
          } else {
            const float sg = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(x[c] * P.neg_al2e));
            ds[c] = dq_ds(sg, da[8 * hh + c], x[c], P.alpha);
          }
        }
        if (kt == last) {
#pragma unroll
          for (int c = 0; c < 8; ++c)
            if (j0 + c_row(8 * hh + c, g) > i) ds[c] = 0.0f;
        }
        sm.p[b][w][hh][lane] = pack8(ds);
      }
    }
    lds_barrier();
    const int x0 = first64 ? (par ? S_WAVES : 0) : par, dx = first64 ? 1 : 2;
    for (int x = x0; x < S_WAVES; x += dx)
      if (k0 + x <= last) accumulate_from<D>(sm.x[x][b], sm.p[b][x], db0, g, lane, acc);
  }
  lds_barrier();
  put_sums<D>(sm.red[par], acc, db0, l32, g);
  lds_barrier();
  const int64_t at = (e.start + i0) * P.out_stride + h * D;
  emit_rows<D, true>(sm.red[0], tid, P.dq + at, P.out_stride, e.len - i0,
                     first64 ? P.dk_scale_l2 : P.dqk_scale, P.h_dq ? P.h_dq + at : nullptr);
}

// `hist`: the item's d_time sums, [nb][2^time_cs].
template <int D, bool POS, bool TIME, bool DET>
__device__ __forceinline__ void short_dkv(const SParams &P, ShortBwdSmem<D, DET> &sm,
                                          typename TabAcc<DET>::L *hist, int item) {
  typedef TabAcc<DET> A;
  WorkEntry e;
  int h, j0;
  if (!short_item(P, P.list_k, item, e, h, j0)) return;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = j0 + l32, first = j0 / ST, tiles = (e.len + ST - 1) / ST;
  // What this wave accumulates, in the tile kernels' order.  d = 64: dV and dK
  // of half the dims over the even or the odd tiles (par), which are added at
  // the end; d = 128: one of the two (par) for half the dims over every tile.
  constexpr bool SPLIT = D == 128;
  constexpr int NB = D / 64;
  const int par = w & 1, db0 = NB * (w >> 1);
  u16 *qs = sm.x[w][0], *os = sm.x[w][1];
  const __amdgpu_buffer_rsrc_t rq = head_rows<D>(P, P.q, e, h), ro = head_rows<D>(P, P.dO, e, h),
                               rp = pos_table(P, POS, h);
  Rows<D> qr, dr, kr, vr;
  qr.load(P, rq, j0 + ST * w + l32, g);
  kr.load(P, head_rows<D>(P, P.k, e, h), j, g);
  dr.load(P, ro, j0 + ST * w + l32, g);
  vr.load(P, head_rows<D>(P, P.v, e, h), j, g);
  float pw[16];
  if (POS) load_pos<-1>(P, rp, j - (j0 + ST * w + 4 * g), pw);
  TimeAxis ax{};
  int64_t tq = 0;
  if (TIME) {
    tq = ts_of(P, e, j0 + ST * w + l32);
    ax.set(P, e, j);
    for (int x = tid; x < P.nb << P.time_cs; x += S_THREADS) hist[x] = 0;
    stage_table(P, sm.t, h, tid, P.inv_alpha);
  }
  if (POS) {
    sm.win[w][0][lane] = 0;
    sm.win[w][1][lane] = 0;
  }
  if (TIME) __syncthreads();
  typename A::L *my_t = hist + (lane & ((1 << P.time_cs) - 1));
  typename A::G *dp = POS ? (typename A::G *)P.dpos_part + e.start * P.H + h : nullptr;
  TimeRun<A> run;
  f32x16 dv[NB], dk[SPLIT ? 1 : NB];            // (SPLIT: dV or dK, in dv)
  clear(dv);
  clear(dk);

  for (int q0 = first; q0 < tiles; q0 += S_WAVES) {
    const int qt = q0 + w, i0 = ST * qt, ni = i0 + ST * S_WAVES;
    if (q0 > first) lds_barrier();              // the step before is read
    if (qt < tiles) {
      qr.store(qs, l32, g);
      dr.store(os, l32, g);
      const bool slow = TIME && ax.stage(sm.t.rel[w], tq, lane);
      if (TIME) wave_lds_fence();
      f32x16 s, da;
#pragma unroll
      for (int r = 0; r < 16; ++r) { s[r] = POS ? pw[r] * P.inv_alpha : 0.0f; da[r] = 0.0f; }
      s = score<D>(qr, kr, s);
      da = score<D>(dr, vr, da);
      if (qt + S_WAVES < tiles) {
        qr.load(P, rq, ni + l32, g);
        dr.load(P, ro, ni + l32, g);
        if (POS) load_pos<-1>(P, rp, j - (ni + 4 * g), pw);
        if (TIME) tq = ts_of(P, e, ni + l32);
      }
      float carry = 0.0f;       // d_pos: a quad's row-head sums for the next quad
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        float x[8], a[8], ds[8];
        int tk[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) x[c] = s[8 * hh + c];
        if (TIME) {
          if (!slow) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
              const float4 t4 = *(const float4 *)(sm.t.rel[w] + 16 * hh + 8 * q + 4 * g);
              tk[4 * q + 0] = time_index(t4.x - ax.own_rel);
              tk[4 * q + 1] = time_index(t4.y - ax.own_rel);
              tk[4 * q + 2] = time_index(t4.z - ax.own_rel);
              tk[4 * q + 3] = time_index(t4.w - ax.own_rel);
            }
#pragma unroll
            for (int c = 0; c < 8; ++c) x[c] += sm.t.tab[tk[c]];
          } else {
#pragma unroll
            for (int c = 0; c < 8; ++c) {
              const int64_t gap = ts_of(P, e, i0 + c_row(8 * hh + c, g)) - ax.own;
              tk[c] = time_bucket(gap, P.nb);
              x[c] += far_time(P, h, gap, P.inv_alpha);
            }
          }
        }
        // A and dS times log2e
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          const float u = x[c] * P.al2e;
          const float sg = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-u));
          a[c] = u * sg;
          ds[c] = dkv_ds(a[c], sg, da[8 * hh + c]);
        }
        // query rows past the sequence have dO = 0: only the diagonal tile needs
        // the causal mask (keys past the sequence lie in it alone)
        if (qt == first) {
#pragma unroll
          for (int c = 0; c < 8; ++c)
            if (i0 + c_row(8 * hh + c, g) < j) { a[c] = 0.0f; ds[c] = 0.0f; }
        }
        if constexpr (POS) {
          // slot i - j + 31 (- the tile's offset); summed along the diagonals as in
          // the tile kernels' dK/dV items.  (A function for both: the tile kernels
          // up to 1% slower, scheduled otherwise.)
          typename A::L *pd = &sm.win[w][g][4 * g + ST - 1 - l32];
          const bool row_head = (lane & 15) < 3;
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const float *v = ds + 4 * q;
            const float b4 = ((v[0] + row_shl<1>(v[1])) + row_shl<2>(v[2])) + row_shl<3>(v[3]);
            const float band = hh == 0 && q == 0 ? b4 : b4 + carry;
            const float head = (v[3] + row_shr<1>(v[2])) + row_shr<2>(v[1]);
            const int at = 16 * hh + 8 * q;
            atomicAdd(pd + at, A::lds(band));
            if (hh == 1 && q == 1) {
              if (row_head) atomicAdd(pd + at + 3, A::lds(head));
            } else {
              carry = row_shr<5>(row_head ? head : 0.0f);
            }
          }
        }
        if (TIME) {
          if (!slow) {
            if (hh == 0) run.start(tk[0]);
#pragma unroll
            for (int c = 0; c < 8; ++c) run.add(my_t, P.nb, P.time_cs, tk[c], ds[c]);
          } else {
#pragma unroll
            for (int c = 0; c < 8; ++c)
              if (ds[c] != 0.0f) atomicAdd(&my_t[tk[c] << P.time_cs], A::lds(ds[c]));
          }
        }
        sm.p[0][w][hh][lane] = pack8(a);
        sm.p[1][w][hh][lane] = pack8(ds);
      }
      if constexpr (POS) {
        // the tile's 63 diagonals to the sequence's partials
        wave_lds_fence();
        const typename A::L v = sm.win[w][0][lane] + sm.win[w][1][lane];
        sm.win[w][0][lane] = 0;
        sm.win[w][1][lane] = 0;
        const int m = i0 - j0 + lane - (ST - 1);
        if (v != 0 && m >= 0 && m < e.len) atomicAdd(&dp[(int64_t)m * P.H], A::glob(v));
      }
    }
    lds_barrier();
    if constexpr (SPLIT) {
      for (int x = 0; x < S_WAVES; ++x)
        if (q0 + x < tiles)
          accumulate_from<D>(sm.x[x][par ? 0 : 1], sm.p[par][x], db0, g, lane, dv);
    } else {
      for (int x = (par ^ q0) & 1; x < S_WAVES; x += 2)
        if (q0 + x < tiles) {
          accumulate_from<D>(sm.x[x][1], sm.p[0][x], db0, g, lane, dv);
          accumulate_from<D>(sm.x[x][0], sm.p[1][x], db0, g, lane, dk);
        }
    }
  }
  if (TIME) run.flush(my_t, P.nb, P.time_cs);
  lds_barrier();
  put_sums<D>(sm.red[par], dv, db0, l32, g);
  if constexpr (!SPLIT) put_sums<D>(sm.red[2 + par], dk, db0, l32, g);
  lds_barrier();
  const int64_t at = (e.start + j0) * P.out_stride + h * D;
  emit_rows<D, !SPLIT>(sm.red[SPLIT ? 1 : 2], tid, P.dk + at, P.out_stride, e.len - j0,
                       P.dk_scale_l2, P.h_dk ? P.h_dk + at : nullptr);
  emit_rows<D, !SPLIT>(sm.red[0], tid, P.dv + at, P.out_stride, e.len - j0, P.dv_scale_l2,
                       P.h_dv ? P.h_dv + at : nullptr);
  if (TIME) {
    typename A::GT *part = (typename A::GT *)P.dtime_part +
                          ((int64_t)(item % DTIME_BINS) * P.H + h) * P.nb;
    for (int x = tid; x < P.nb; x += S_THREADS) {
      typename A::L v = 0;
      for (int c = 0; c < 1 << P.time_cs; ++c) v += hist[(x << P.time_cs) + c];
      if (v != 0) atomicAdd(&part[x], (typename A::GT)v);
    }
  }
}

// Both item kinds of the backward in one launch, in turn down the
// longest-first lists.
template <int D, bool POS, bool TIME, bool DET>
__global__ void __launch_bounds__(S_THREADS, D == 64 ? 2 : 1) short_bwd_kernel(SParams P) {
  __shared__ __attribute__((aligned(16))) ShortBwdSmem<D, DET> sm;
  extern __shared__ double dyn_short[];
  if (blockIdx.x & 1) short_dq<D, POS, TIME, DET>(P, sm, blockIdx.x >> 1);
  else short_dkv<D, POS, TIME, DET>(P, sm, (typename TabAcc<DET>::L *)dyn_short, blockIdx.x >> 1);
}

SParams make_params(const AttnArgs &a) {
  char *ws = (char *)a.ws;
  SParams P{};
  P.q = (const u16 *)a.q;
  P.k = (const u16 *)a.k;
  P.v = (const u16 *)a.v;
  P.pos_w = a.pos_w;
  P.time_w = a.time_w;
  P.ts = a.ts;
  P.off = a.off;
  P.ctrl = (int32_t *)(ws + a.L.ctrl);
  P.list_q = (const WorkEntry *)(ws + a.L.list_q);
  P.list_k = (const WorkEntry *)(ws + a.L.list_k);
  P.T = a.p.T;
  P.B = a.p.B;
  P.H = a.p.H;
  P.N = a.p.N;
  P.nb = a.p.has_time ? a.p.nb : 0;
  P.out_stride = a.p.H * a.p.d;
  P.time_cs = hist_copies_log2(P.nb);
  P.alpha = a.p.alpha;
  P.inv_alpha = 1.0f / a.p.alpha;
  P.neg_al2e = -a.p.alpha * L2E;
  P.al2e = a.p.alpha * L2E;
  P.dqk_scale = a.p.alpha / (float)a.p.N;
  P.dk_scale_l2 = P.dqk_scale / L2E;
  P.dv_scale_l2 = 1.0f / (float)a.p.N / L2E;
  return P;
}

template <int D>
auto pick_fwd(bool pos, bool time) {
  return pos ? (time ? short_fwd_kernel<D, true, true> : short_fwd_kernel<D, true, false>)
             : (time ? short_fwd_kernel<D, false, true> : short_fwd_kernel<D, false, false>);
}
template <int D, bool DET>
auto pick_bwd(bool pos, bool time) {
  return pos ? (time ? short_bwd_kernel<D, true, true, DET> : short_bwd_kernel<D, true, false, DET>)
             : (time ? short_bwd_kernel<D, false, true, DET>
                     : short_bwd_kernel<D, false, false, DET>);
}

}  // namespace

// The line: the batch's work-groups all run at once (the forward has one
// work-group per 32-row item and room for three on a compute unit at d = 64,
// the backward two per item and room for two; one at d = 128, where a second
// gains nothing).  Then a call is as long as its longest chain, and
// the chain here is the shorter one.  Beyond it the items queue, each with its
// exposed start, where the tile kernels' persistent work-groups hide theirs.
// Tile kernels / these, both biases, H = 4 where not said (us):
//   forward d = 64:  B=1 L=502 16.2 / 11.7, B=1 L=812 21.8 / 15.3, B=1 L=8022 H=2
//     148 / 110, B=12 L<=250 10.7 / 8.9, B=4 L<=1630 28.5 / 24.4; past it B=12
//     L<=1000 26.7 / 27.9, B=32 L<=300 15.3 / 17.9
//   forward d = 128: B=1 L=502 19.9 / 16.5, B=4 L<=512 18.4 / 16.0, B=1 L=2000 H=1
//     53.8 / 37.7; past it B=12 L<=250 14.3 / 14.0
//   backward d = 64: B=1 L=90 23.3 / 16.3, B=1 L=812 57.9 / 39.1, B=4 L<=512 42.6 /
//     28.4, B=32 L<=100 H=2 23.4 / 19.2; past it B=32 L<=300 38.0 / 51.1, B=12 L<=1000
//     68.5 / 78.5
//   backward d = 128: B=1 L=502 45.3 / 33.9, B=1 L=2000 H=1 123 / 85, B=4 L<=512 H=2
//     44.1 / 32.3; past it B=12 L<=250 34.3 / 38.6
static int64_t short_items(const Problem &p) { return 2 * p.max_entries * p.H; }

bool fwd_short(const Problem &p, int dev) {
  return p.dtype == HSTU_BF16 &&
         short_items(p) <= (p.d == 64 ? 3 : 1) * (int64_t)device_info(dev).num_cu;
}
bool bwd_short(const Problem &p, int dev) {
  return p.dtype == HSTU_BF16 &&
         2 * short_items(p) <= (p.d == 64 ? 2 : 1) * (int64_t)device_info(dev).num_cu;
}

hipError_t launch_attn_fwd_short(const AttnArgs &a, void *o, bool direct, hipStream_t s) {
  SParams P = make_params(a);
  P.o = (u16 *)o;
  P.direct = direct ? 1 : 0;
  auto kfn = a.p.d == 64 ? pick_fwd<64>(a.p.has_pos, a.p.has_time)
                         : pick_fwd<128>(a.p.has_pos, a.p.has_time);
  hipLaunchKernelGGL(kfn, dim3((unsigned)(2 * a.p.max_entries * a.p.H)), dim3(S_THREADS), 0, s, P);
  return hipGetLastError();
}

hipError_t launch_attn_bwd_short(const AttnArgs &a, const void *dO, void *dq, void *dk, void *dv,
                                 const GradOut *go, hipStream_t s) {
  const char *ws = (const char *)a.ws;
  const Problem &p = a.p;
  SParams P = make_params(a);
  P.dO = (const u16 *)dO;
  P.dq = (u16 *)dq;
  P.dk = (u16 *)dk;
  P.dv = (u16 *)dv;
  if (go) {
    P.out_stride = go->stride;
    P.h_dq = (const u16 *)go->h_dq;
    P.h_dk = (const u16 *)go->h_dk;
    P.h_dv = (const u16 *)go->h_dv;
  }
  P.dpos_part = a.L.dpos_part ? (void *)(ws + a.L.dpos_part) : nullptr;
  P.dtime_part = a.L.dtime_part ? (void *)(ws + a.L.dtime_part) : nullptr;
  auto kfn = p.d == 64 ? (p.deterministic ? pick_bwd<64, true>(p.has_pos, p.has_time)
                                          : pick_bwd<64, false>(p.has_pos, p.has_time))
                       : (p.deterministic ? pick_bwd<128, true>(p.has_pos, p.has_time)
                                          : pick_bwd<128, false>(p.has_pos, p.has_time));
  hipLaunchKernelGGL(kfn, dim3((unsigned)(4 * p.max_entries * p.H)), dim3(S_THREADS),
                     p.has_time ? sizeof(double) * (size_t)P.nb << P.time_cs : 0, s, P);
  return hipGetLastError();
}

}  // namespace hstu
