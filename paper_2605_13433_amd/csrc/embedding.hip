// Jagged multi-table embedding lookup for gfx950 (Sec. 4.1.2, "Jagged
// Embedding Lookup Acceleration"): explicit jagged indices (table offsets,
// no padding ids) and table-grouped work distribution.
//
// Forward: a gather of 16-byte row chunks.  The ids are table-major and
// every work-group takes a contiguous run of them, so the grid sweeps the
// tables one after the other and all compute units work on the same one or
// two tables at any time: a hot table's rows are fetched into each XCD's L2
// once and reused by every work-group there.  Rows land either flat
// ([num_ids][D]) or straight in the token-major concatenated layout
// ([T][F*D]) that a sequence model consumes, so no conversion pass follows.
//
// Backward: deterministic sparse gradient.  Each id becomes its global row
// key (row_offsets[t] + id; invalid ids get a sentinel that sorts last; 32
// bits while the rows fit, which halves what the sort moves); a stable radix
// sort orders the positions by key; head counts per chunk number the distinct
// rows; then fixed 32-position chunks of the sorted order sum the
// output-gradient rows of each distinct key in position order, writing rows
// that start and end inside a chunk directly and chunk-boundary pieces as
// partials that are joined in chunk order (within a chunk work-group by
// itself, across work-groups by a fix-up pass).  Every sum has a
// fixed order, so the result is bitwise reproducible (no float atomics),
// and a hot row that occurs thousands of times is summed by many chunks in
// parallel instead of by one serial loop.
//
// Measured on 8 tables of 2^22 .. 2^7 rows, 77 971 ids each, D = 128, fp32:
// backward 265 -> 218 us where the forward ran just before it (chunk pass 133,
// keys 6, sort with its clears 62, rows' numbering 8, fix-up 9.5), 187 us by
// itself (chunk pass 104, the others the same).  The chunk pass reads 319 MB of
// gradients: plain loads of those bytes take 66 us from clean memory and
// 111-130 us behind 1 GiB of dirty lines, in sorted or sequential order alike.
// Sort passes 25 -> 15 us each, fix-up 29 -> 9, the rows' numbering 17 -> 8.
// Non-temporal forward stores changed nothing.  bf16, backward by itself: 130
// (chunk pass 49).
#include <rocprim/device/device_radix_sort.hpp>

#include <algorithm>

#include "internal.h"
#include "device.h"
#include "../../include/hstu_embedding.h"

namespace hstu {
namespace {

constexpr int ET = 256;             // threads per work-group
constexpr int FWD_UNROLL = 4;       // 16-byte chunks in flight per thread
constexpr int CHUNK = 32;           // sorted positions per backward chunk
constexpr int MAX_TABLES = 1024;
constexpr int BWD_UNROLL = 8;       // gradient rows in flight per thread
constexpr int MAX_CPB = 16;         // backward chunks per work-group
constexpr int FIX_UNROLL = 8;       // group pieces in flight per thread of the join

// Threads per chunk and chunks per work-group of the backward chunk pass
// for `cpr` 16-byte slices per row (host and device agree on this).
__host__ __device__ __forceinline__ int chunk_tpc(int cpr) { return cpr < ET ? cpr : ET; }
__host__ __device__ __forceinline__ int chunk_cpb(int cpr) {
  const int c = ET / chunk_tpc(cpr);
  return c < MAX_CPB ? c : MAX_CPB;
}

// 16-byte vector of the row element type: 4 floats or 8 bf16.
template <typename T> struct Elt;
template <> struct Elt<float> { static constexpr int N = 4; };
template <> struct Elt<u16> { static constexpr int N = 8; };

__device__ __forceinline__ void add_chunk(float *acc, const uint4 &v, float) {
  acc[0] += __uint_as_float(v.x);
  acc[1] += __uint_as_float(v.y);
  acc[2] += __uint_as_float(v.z);
  acc[3] += __uint_as_float(v.w);
}
__device__ __forceinline__ void add_chunk(float *acc, const uint4 &v, u16) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    acc[2 * i] += __uint_as_float(w[i] << 16);
    acc[2 * i + 1] += __uint_as_float(w[i] & 0xffff0000u);
  }
}

// Table of id position r: the last t with id_offsets[t] <= r (empty tables
// are skipped because their successor has the same offset).
__device__ __forceinline__ int table_of(const int64_t *io, int F, int64_t r) {
  int lo = 0, hi = F - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (io[mid] <= r) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Table of id position r under the call's layout: in the token layout every
// table holds per_table ids, so the table follows from r alone (never from
// the offsets array, which keeps every output address in bounds whatever
// that array holds).
__device__ __forceinline__ int table_at(bool token, const int64_t *io, int F, int64_t r,
                                        int64_t per_table) {
  // (32-bit: num_ids < 2^31)
  return token ? (int)((uint32_t)r / (uint32_t)per_table) : table_of(io, F, r);
}

// Global row of id `id` in table t, or -1 if the id lies outside its table
// (or the table outside the weight matrix).
__device__ __forceinline__ int64_t global_row(const int64_t *ro, int t, int64_t id,
                                              int64_t total_rows) {
  const int64_t g = ro[t] + id;
  return (id >= 0 && id < ro[t + 1] - ro[t] && ro[t] >= 0 && g < total_rows) ? g : -1;
}

// Where row chunk c of id position r (table t) goes in the output layout.
__device__ __forceinline__ int64_t out_elem(bool token, int64_t r, int t, const int64_t *io,
                                            int F, int D, int64_t per_table, int c, int n_e) {
  return token ? (r - (int64_t)t * per_table) * ((int64_t)F * D) + (int64_t)t * D + c * n_e
               : r * D + c * n_e;
}

struct FwdArgs {
  const void *w;
  const int64_t *ro, *io, *ids;
  void *out;
  int64_t n, per_table, total_rows;
  int F, D, rows_per_block;
  bool token;
};

// Block b gathers id positions [b*RB, (b+1)*RB): thread x handles local
// chunks x, x+ET, ... of those rows (chunk = 16 bytes of a row).
template <typename T>
__global__ void __launch_bounds__(ET) emb_fwd_kernel(FwdArgs a) {
  __shared__ int64_t s_io[MAX_TABLES + 1], s_ro[MAX_TABLES + 1];
  constexpr int NE = Elt<T>::N;
  for (int i = threadIdx.x; i <= a.F; i += ET) {
    s_io[i] = a.io[i];
    s_ro[i] = a.ro[i];
  }
  __syncthreads();
  const int cpr = a.D / NE;
  const int64_t r0 = (int64_t)blockIdx.x * a.rows_per_block;
  const int local = a.rows_per_block * cpr;
  const T *W = (const T *)a.w;
  T *out = (T *)a.out;
  uint4 v[FWD_UNROLL];
  int64_t dst[FWD_UNROLL];
#pragma unroll
  for (int k = 0; k < FWD_UNROLL; ++k) {
    const int x = threadIdx.x + k * ET;
    dst[k] = -1;
    v[k] = make_uint4(0, 0, 0, 0);
    if (x < local) {
      const int64_t r = r0 + x / cpr;
      const int c = x % cpr;
      if (r < a.n) {
        const int t = table_at(a.token, s_io, a.F, r, a.per_table);
        const int64_t g = global_row(s_ro, t, a.ids[r], a.total_rows);
        if (g >= 0) v[k] = *(const uint4 *)(W + g * a.D + c * NE);
        dst[k] = out_elem(a.token, r, t, s_io, a.F, a.D, a.per_table, c, NE);
      }
    }
  }
#pragma unroll
  for (int k = 0; k < FWD_UNROLL; ++k)
    if (dst[k] >= 0) *(uint4 *)(out + dst[k]) = v[k];
}

// ---------------------------------------------------------------- backward
constexpr int HEAD_BLOCK = 4096;    // sorted positions per head-count block (128 chunks)
// The blocks' head counts are summed by every chunk work-group for itself up
// to this many (2 M positions), by a scan launch above.
constexpr int HEAD_SUM_BLOCKS = 512;

// State of a chunk, and of a group of chunks for the fix-up pass.
enum : uint32_t {
  CHUNK_INSIDE = 1,                 // all its positions belong to one row that began
                                    // before it and goes on after it
  CHUNK_STARTS = 2,                 // a row begins in it and goes on after it
  CHUNK_HEAD = 4                    // its first row began before it
};

template <typename K>
struct BwdArgs {
  const int64_t *ro, *io, *ids;
  const void *dout;
  float *grad;
  int64_t *unique_rows;
  int32_t *num_unique;
  K *keys_in, *keys;
  uint32_t *pos_in, *pos;
  uint32_t *chunk_heads;             // [nchunks]: distinct rows that begin in the chunk
  uint32_t *block_heads;             // [nblocks]: in the block; scanned: before it
  // per group of `cpb` chunks (a chunk work-group's)
  uint32_t *state;                   // [ngroups]: CHUNK_* bits
  float *part;                       // [ngroups][2][D]: first, last piece
  K sentinel;                        // total_rows
  int64_t n, per_table;
  int F, D, nchunks, nblocks, ngroups;
  bool token, scanned;
};

template <typename K>
__global__ void __launch_bounds__(ET) emb_keys_kernel(BwdArgs<K> a) {
  __shared__ int64_t s_io[MAX_TABLES + 1], s_ro[MAX_TABLES + 1];
  for (int i = threadIdx.x; i <= a.F; i += ET) {
    s_io[i] = a.io[i];
    s_ro[i] = a.ro[i];
  }
  __syncthreads();
  const int64_t r = (int64_t)blockIdx.x * ET + threadIdx.x;
  if (r >= a.n) return;
  const int t = table_at(a.token, s_io, a.F, r, a.per_table);
  const int64_t g = global_row(s_ro, t, a.ids[r], (int64_t)a.sentinel);
  a.keys_in[r] = g >= 0 ? (K)g : a.sentinel;
  a.pos_in[r] = (uint32_t)r;
}

// Whether a distinct row begins at sorted position p (< n).
template <typename K>
__device__ __forceinline__ bool head_at(const BwdArgs<K> &a, int64_t p) {
  const K k = a.keys[p];
  return k != a.sentinel && (p == 0 || a.keys[p - 1] != k);
}

// Rows that begin in each chunk and in each block of HEAD_BLOCK positions.
template <typename K>
__global__ void __launch_bounds__(ET) emb_heads_kernel(BwdArgs<K> a) {
  constexpr int ROUNDS = HEAD_BLOCK / ET;
  __shared__ uint32_t total;
  const int lane = threadIdx.x & 63;
  if (threadIdx.x == 0) total = 0;
  __syncthreads();
  const int64_t p0 = (int64_t)blockIdx.x * HEAD_BLOCK;
  uint32_t mine = 0;
#pragma unroll
  for (int x = 0; x < ROUNDS; ++x) {
    const int64_t p = p0 + x * ET + threadIdx.x;
    const uint64_t heads = __ballot(p < a.n && head_at(a, p));
    // a wave's 64 positions are two chunks
    const uint32_t c = __popc((uint32_t)(lane < 32 ? heads : heads >> 32));
    if ((lane & 31) == 0 && p < a.n) a.chunk_heads[p / CHUNK] = c;
    mine += lane == 0 || lane == 32 ? c : 0u;
  }
  if (mine) atomicAdd(&total, mine);
  __syncthreads();
  if (threadIdx.x == 0) a.block_heads[blockIdx.x] = total;
}

// block_heads -> sums over the blocks before (many blocks only): one
// work-group, a contiguous share of the blocks a thread.
template <typename K>
__global__ void __launch_bounds__(1024) emb_scan_kernel(BwdArgs<K> a) {
  __shared__ uint32_t part[1024];
  const int64_t per = (a.nblocks + 1023) / 1024, b0 = threadIdx.x * per;
  const int64_t b1 = b0 + per < a.nblocks ? b0 + per : a.nblocks;
  uint32_t s = 0;
  for (int64_t b = b0; b < b1; ++b) s += a.block_heads[b];
  part[threadIdx.x] = s;
  __syncthreads();
  uint32_t before = 0;
  for (int x = 0; x < (int)threadIdx.x; ++x) before += part[x];
  for (int64_t b = b0; b < b1; ++b) {
    const uint32_t c = a.block_heads[b];
    a.block_heads[b] = before;
    before += c;
  }
}

// Output-gradient element offset of chunk c of id position r.
template <typename K>
__device__ __forceinline__ int64_t dout_elem(const BwdArgs<K> &a, uint32_t r, int c, int n_e) {
  if (!a.token) return (int64_t)r * a.D + c * n_e;
  const uint32_t t = r / (uint32_t)a.per_table;       // num_ids < 2^31
  return (int64_t)(r - t * (uint32_t)a.per_table) * ((int64_t)a.F * a.D) +
         (int64_t)t * a.D + c * n_e;
}

// NE floats to 16-byte aligned memory.
template <int NE>
__device__ __forceinline__ void store_slice(float *dst, const float (&acc)[NE]) {
#pragma unroll
  for (int e = 0; e < NE; e += 4)
    *(float4 *)(dst + e) = make_float4(acc[e], acc[e + 1], acc[e + 2], acc[e + 3]);
}

// One chunk of CHUNK sorted positions per group of `tpc` threads; a thread
// sums its 16-byte column slices over the chunk's pieces (runs of equal
// key) in position order; the pieces that cross chunks are joined in chunk
// order within the work-group, so that only what crosses work-groups is left
// to the fix-up pass (a row of 15 891 positions: 62 pieces instead of 497).
// Bound by the gradient rows' reads: everything the
// loop needs besides them (keys, row offsets, the rows' ranks) is in LDS
// before it, since a wait for any other load would also wait for the rows in
// flight.
template <typename T, typename K>
__global__ void __launch_bounds__(ET) emb_chunk_kernel(BwdArgs<K> a) {
  constexpr int NE = Elt<T>::N;
  const int cpr = a.D / NE;
  const int tpc = chunk_tpc(cpr), cpb = chunk_cpb(cpr);
  __shared__ K s_key[MAX_CPB * CHUNK];
  __shared__ int64_t s_row[MAX_CPB * CHUNK];           // element offset of the gradient row
  __shared__ uint32_t s_rank[MAX_CPB * CHUNK];         // distinct rows up to the position
  __shared__ uint32_t s_sum[ET / 64], s_wave[MAX_CPB * CHUNK / 64], s_state[MAX_CPB];
  __shared__ __attribute__((aligned(16))) float s_part[2][ET * NE];   // cpb > 1: chunk g's
                                                                     // pieces at g D
  const int tid = threadIdx.x, lane = tid & 63;
  const int g = tid / tpc, lt = tid % tpc;
  const int64_t chunk0 = (int64_t)blockIdx.x * cpb, chunk = chunk0 + g;
  const int64_t p0 = chunk * CHUNK;
  // stage the keys and rows of this block's chunks and number their heads
  const int npos = cpb * CHUNK;                        // at most 2 a thread
  for (int i = tid; i < (npos + 63) / 64 * 64; i += ET) {
    const int64_t p = chunk0 * CHUNK + i;
    const bool in = i < npos && p < a.n;
    const bool head = in && head_at(a, p);
    const uint64_t heads = __ballot(head);
    if (i < npos) {
      s_key[i] = in ? a.keys[p] : a.sentinel;
      s_row[i] = in ? dout_elem(a, a.pos[p], 0, NE) : 0;
      s_rank[i] = __popcll(heads & (~0ull >> (63 - lane)));      // heads up to this lane
    }
    if (lane == 0) s_wave[i / 64] = __popcll(heads);
  }
  // distinct rows before the block's first position
  const int64_t blk = chunk0 / (HEAD_BLOCK / CHUNK);
  uint32_t before = 0;
  if (a.scanned) before = tid == 0 ? a.block_heads[blk] : 0u;
  else for (int64_t b = tid; b < blk; b += ET) before += a.block_heads[b];
  for (int64_t c = blk * (HEAD_BLOCK / CHUNK) + tid; c < chunk0; c += ET)
    before += a.chunk_heads[c];
  before = (uint32_t)wave_prefix((int32_t)before);
  if (lane == 63) s_sum[tid >> 6] = before;
  __syncthreads();
  uint32_t base = 0;
#pragma unroll
  for (int x = 0; x < ET / 64; ++x) base += s_sum[x];
  if (blockIdx.x == gridDim.x - 1 && tid == 0 && a.num_unique) {
    uint32_t all = base;
    for (int x = 0; x < (npos + 63) / 64; ++x) all += s_wave[x];
    *a.num_unique = (int32_t)all;
  }
  // heads in the waves' spans before this chunk's
  for (int x = 0; x < g * CHUNK / 64 && g < cpb; ++x) base += s_wave[x];
  const K *key = s_key + g * CHUNK;
  const int64_t *row = s_row + g * CHUNK;
  const uint32_t *rank = s_rank + g * CHUNK;
  const int pe = g < cpb && chunk < a.nchunks ? (int)std::min<int64_t>(CHUNK, a.n - p0) : 0;
  // sorted: the sentinel keys (invalid ids) form the array's tail
  int valid = 0;
  while (valid < pe && key[valid] != a.sentinel) ++valid;
  const bool prev_same = valid > 0 && p0 > 0 && a.keys[p0 - 1] == key[0];
  const bool next_same =
      valid > 0 && valid == pe && p0 + pe < a.n && a.keys[p0 + pe] == key[pe - 1];
  if (lt == 0 && g < cpb) {
    const bool one = valid > 0 && key[0] == key[valid - 1];
    s_state[g] = (prev_same ? CHUNK_HEAD : 0u) |
                 (next_same ? (one && prev_same ? CHUNK_INSIDE : CHUNK_STARTS) : 0u);
  }
  const T *G = (const T *)a.dout;
  for (int c = lt; c < cpr && valid > 0; c += tpc) {
    float acc[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) acc[e] = 0.0f;
    int start = 0;
    for (int q0 = 0; q0 < valid; q0 += BWD_UNROLL) {
      uint4 v[BWD_UNROLL];
#pragma unroll
      for (int u = 0; u < BWD_UNROLL; ++u)
        v[u] = q0 + u < valid ? *(const uint4 *)(G + row[q0 + u] + c * NE)
                              : make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int u = 0; u < BWD_UNROLL; ++u) {
        const int q = q0 + u;
        if (q >= valid) break;
        add_chunk(acc, v[u], T{});
        const K k = key[q];
        if (q + 1 < valid && key[q + 1] == k) continue;
        // piece [start, q] of key k ends here
        const bool first = start > 0 || !prev_same;
        const bool last = q + 1 < valid || !next_same;
        const int slot = first ? 1 : 0;
        if (first && last) store_slice<NE>(a.grad + (uint64_t)k * (uint64_t)a.D + c * NE, acc);
        else if (cpb > 1) store_slice<NE>(s_part[slot] + g * a.D + c * NE, acc);
        else store_slice<NE>(a.part + (chunk * 2 + slot) * a.D + c * NE, acc);
        if (first && c == 0 && a.unique_rows)
          a.unique_rows[base + rank[start] - 1] = (int64_t)k;
#pragma unroll
        for (int e = 0; e < NE; ++e) acc[e] = 0.0f;
        start = q + 1;
      }
    }
  }
  __syncthreads();
  if (cpb == 1) {
    if (tid == 0) a.state[blockIdx.x] = s_state[0];
    return;
  }
  // join: the group of the chunk a row starts in (or of the work-group's first
  // chunk, for a row that began before) adds the pieces of the chunks after
  // it; slices of one thread each (cpb > 1: cpr = tpc).  What does not end in
  // the work-group is its first (slot 0) or last (slot 1) piece.
  const int chunks = (int)std::min<int64_t>(cpb, a.nchunks - chunk0);
  if (g < chunks) {
    const uint32_t st = s_state[g];
#pragma unroll
    for (int slot = 0; slot < 2; ++slot) {
      if (slot == 0 ? !(g == 0 && (st & CHUNK_HEAD)) : !(st & CHUNK_STARTS)) continue;
      float acc[NE];
#pragma unroll
      for (int e = 0; e < NE; ++e) acc[e] = s_part[slot][g * a.D + lt * NE + e];
      bool open = slot == 1 || (st & CHUNK_INSIDE);
      for (int j = g + 1; j < chunks && open; ++j) {
#pragma unroll
        for (int e = 0; e < NE; ++e) acc[e] += s_part[0][j * a.D + lt * NE + e];
        open = s_state[j] & CHUNK_INSIDE;
      }
      if (slot == 1 && !open) {
        const K k = key[CHUNK - 1];
        store_slice<NE>(a.grad + (uint64_t)k * (uint64_t)a.D + lt * NE, acc);
      } else {
        store_slice<NE>(a.part + ((int64_t)blockIdx.x * 2 + slot) * a.D + lt * NE, acc);
      }
    }
  }
  if (tid == 0) {
    // the work-group as one chunk: its last chunk that is not all inside one
    // row decides
    uint32_t st = s_state[0] & CHUNK_HEAD;
    int j = chunks - 1;
    while (j >= 0 && (s_state[j] & CHUNK_INSIDE)) --j;
    if (j < 0) st |= CHUNK_INSIDE;
    else if (s_state[j] & CHUNK_STARTS) st |= CHUNK_STARTS;
    a.state[blockIdx.x] = st;
  }
}

// Joins the pieces of rows that cross the chunk groups.  Work-group b serves
// the row (if any) that begins in group b and goes on after it: it finds the
// group it ends in (the first that is not all inside it), splits the groups in
// between into one contiguous range per thread group, sums each range in
// order, and adds the sums to group b's own piece in order -- a fixed order for
// a given batch, with a hot row's groups shared by the whole work-group.
template <typename T, typename K>
__global__ void __launch_bounds__(ET) emb_fixup_kernel(BwdArgs<K> a) {
  constexpr int NE = Elt<T>::N;
  const int64_t chunk = blockIdx.x;
  if (!(a.state[chunk] & CHUNK_STARTS)) return;
  const int cpr = a.D / NE;
  const int tpc = chunk_tpc(cpr), groups = ET / tpc;
  __shared__ float s_sum[ET * NE];
  __shared__ int32_t s_end;
  const K k = a.keys[(chunk + 1) * chunk_cpb(cpr) * CHUNK - 1];   // its last position's
  int64_t c_end = chunk;                            // last group holding key k
  for (;;) {
    if (threadIdx.x == 0) s_end = ET;
    __syncthreads();
    const int64_t c = c_end + 1 + threadIdx.x;
    // (the group after one whose row goes on exists)
    if (c < a.ngroups && !(a.state[c] & CHUNK_INSIDE)) atomicMin(&s_end, (int32_t)threadIdx.x);
    __syncthreads();
    const int e = s_end;
    __syncthreads();
    c_end += e < ET ? e + 1 : ET;
    if (e < ET || c_end + 1 >= a.ngroups) break;
  }
  const int64_t nparts = c_end - chunk;             // groups chunk+1 .. c_end
  const int g = threadIdx.x / tpc, lt = threadIdx.x % tpc;
  const int64_t per = (nparts + groups - 1) / groups;
  const int64_t c_lo = chunk + 1 + g * per;
  const int64_t c_hi = std::min<int64_t>(c_lo + per, c_end + 1);
  // every thread runs the same number of slice rounds (the barriers inside)
  const int rounds = (cpr + tpc - 1) / tpc;
  for (int m = 0; m < rounds; ++m) {
    const int c = lt + m * tpc;
    const bool mine = g < groups && c < cpr;
    float acc[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) acc[e] = 0.0f;
    if (mine) {
      // FIX_UNROLL groups' loads in flight, added in order
      for (int64_t c0 = c_lo; c0 < c_hi; c0 += FIX_UNROLL) {
        float4 x[FIX_UNROLL][NE / 4];
#pragma unroll
        for (int j = 0; j < FIX_UNROLL; ++j)
#pragma unroll
          for (int e = 0; e < NE / 4; ++e)
            x[j][e] = c0 + j < c_hi
                          ? *(const float4 *)(a.part + ((c0 + j) * 2 + 0) * a.D + c * NE + 4 * e)
                          : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
        for (int j = 0; j < FIX_UNROLL; ++j) {
          if (c0 + j >= c_hi) break;
#pragma unroll
          for (int e = 0; e < NE / 4; ++e) {
            acc[4 * e] += x[j][e].x; acc[4 * e + 1] += x[j][e].y;
            acc[4 * e + 2] += x[j][e].z; acc[4 * e + 3] += x[j][e].w;
          }
        }
      }
    }
    __syncthreads();
    if (mine) {
#pragma unroll
      for (int e = 0; e < NE; ++e) s_sum[(g * tpc + lt) * NE + e] = acc[e];
    }
    __syncthreads();
    if (g == 0 && c < cpr) {
      const float *src = a.part + (chunk * 2 + 1) * a.D + c * NE;
#pragma unroll
      for (int e = 0; e < NE; ++e) acc[e] = src[e];
      for (int gi = 0; gi < groups; ++gi)
#pragma unroll
        for (int e = 0; e < NE; ++e) acc[e] += s_sum[(gi * tpc + lt) * NE + e];
      float *dst = a.grad + (uint64_t)k * (uint64_t)a.D + c * NE;
#pragma unroll
      for (int e = 0; e < NE; e += 4)
        *(float4 *)(dst + e) = make_float4(acc[e], acc[e + 1], acc[e + 2], acc[e + 3]);
    }
  }
}

__global__ void emb_count_zero_kernel(int32_t *num_unique) { *num_unique = 0; }

// ------------------------------------------------------------------- host
int check_desc(const hstu_emb_desc *d) {
  if (!d) return fail(HSTU_EINVAL, "desc is NULL");
  if (d->dtype != HSTU_F32 && d->dtype != HSTU_BF16)
    return fail(HSTU_EINVAL, "dtype %d is not HSTU_F32 or HSTU_BF16", (int)d->dtype);
  if (d->num_tables < 0 || d->num_tables > MAX_TABLES)
    return fail(HSTU_EINVAL, "num_tables = %d outside [0, %d]", d->num_tables, MAX_TABLES);
  if (d->dim < 8 || d->dim > 4096 || d->dim % 8)
    return fail(HSTU_EINVAL, "dim = %d is not a multiple of 8 in [8, 4096]", d->dim);
  if (d->num_ids < 0 || d->num_ids >= (int64_t)1 << 31)
    return fail(HSTU_EINVAL, "num_ids = %lld outside [0, 2^31)", (long long)d->num_ids);
  if (d->total_rows < 0 || d->total_rows >= (int64_t)1 << 40)
    return fail(HSTU_EINVAL, "total_rows = %lld outside [0, 2^40)", (long long)d->total_rows);
  if (d->layout != HSTU_EMB_FLAT && d->layout != HSTU_EMB_TOKEN)
    return fail(HSTU_EINVAL, "layout %d is not HSTU_EMB_FLAT or HSTU_EMB_TOKEN",
                (int)d->layout);
  if (d->num_ids > 0 && d->num_tables == 0)
    return fail(HSTU_EINVAL, "num_ids = %lld with no tables", (long long)d->num_ids);
  if (d->layout == HSTU_EMB_TOKEN && d->num_tables > 0 && d->num_ids % d->num_tables)
    return fail(HSTU_EINVAL, "token layout: num_ids = %lld is not a multiple of %d tables",
                (long long)d->num_ids, d->num_tables);
  if (d->num_tables > 0 && (!d->row_offsets || !d->id_offsets))
    return fail(HSTU_EINVAL, "row_offsets and id_offsets must be non-null");
  return HSTU_OK;
}

int elt_n(const hstu_emb_desc *d) { return d->dtype == HSTU_F32 ? 4 : 8; }

// Key bytes: 32 bits while the rows and the sentinel fit.
bool small_keys(const hstu_emb_desc *d) { return d->total_rows < (int64_t)0xffffffff; }

struct BwdLayout {
  size_t keys_in, keys, pos_in, pos, chunk_heads, block_heads, state, part, tmp, tmp_bytes, total;
};

BwdLayout bwd_layout(const hstu_emb_desc *d, size_t tmp_bytes) {
  const size_t n = (size_t)d->num_ids, kb = small_keys(d) ? 4 : 8;
  const size_t nch = (n + CHUNK - 1) / CHUNK, cpb = chunk_cpb(d->dim / elt_n(d));
  const size_t groups = (nch + cpb - 1) / cpb;
  BwdLayout L{};
  size_t o = 0;
  auto take = [&](size_t bytes) { const size_t at = o; o = align_up(o + bytes); return at; };
  L.keys_in = take(kb * n);
  L.keys = take(kb * n);
  L.pos_in = take(4 * n);
  L.pos = take(4 * n);
  L.chunk_heads = take(4 * nch);
  L.block_heads = take(4 * ((n + HEAD_BLOCK - 1) / HEAD_BLOCK));
  L.state = take(4 * groups);
  L.part = take(sizeof(float) * 2 * groups * d->dim);
  L.tmp = take(tmp_bytes);
  L.tmp_bytes = tmp_bytes;
  L.total = o;
  return L;
}

// The sort runs the onesweep radix algorithm at every size above a single
// block (its merge-sort path for mid-size inputs is some twenty small
// launches, latency-bound at the batch sizes here), in blocks of 4096 pairs:
// a pass is as long as the chain of blocks that wait for their predecessors'
// counts, and 1024 threads of 4 pairs take a block's share of it fastest (624
// k pairs, three passes and the rest of the call: 347 us; 256 x 12: 360, 256 x
// 6: 384, the library's choice 388).
using SortConfig = rocprim::radix_sort_config<
    rocprim::default_config, rocprim::default_config,
    rocprim::radix_sort_onesweep_config<rocprim::kernel_config<256, 12>,
                                        rocprim::kernel_config<1024, 4>, 8,
                                        rocprim::block_radix_rank_algorithm::match>,
    0>;

unsigned key_bits(int64_t total_rows) {
  unsigned b = 1;
  while (b < 63 && ((uint64_t)1 << b) <= (uint64_t)total_rows) ++b;
  return b;                          // keys (and the sentinel) are < 2^b
}

// Temporary bytes of the sort.
template <typename K>
hipError_t sort_tmp_bytes(int64_t n, int64_t total_rows, size_t *bytes) {
  return rocprim::radix_sort_pairs<SortConfig>(nullptr, *bytes, (K *)nullptr, (K *)nullptr,
                                               (uint32_t *)nullptr, (uint32_t *)nullptr,
                                               (unsigned)n, 0, key_bits(total_rows));
}
hipError_t lib_tmp_bytes(const hstu_emb_desc *d, size_t *bytes) {
  return small_keys(d) ? sort_tmp_bytes<uint32_t>(d->num_ids, d->total_rows, bytes)
                       : sort_tmp_bytes<uint64_t>(d->num_ids, d->total_rows, bytes);
}

template <typename K>
int bwd_launch(const hstu_emb_desc *desc, const int64_t *ids, const void *dout,
               float *grad_weights, int64_t *unique_rows, int32_t *num_unique, char *ws,
               const BwdLayout &L, hipStream_t s) {
  const int64_t n = desc->num_ids;
  BwdArgs<K> a{};
  a.ro = desc->row_offsets;
  a.io = desc->id_offsets;
  a.ids = ids;
  a.dout = dout;
  a.grad = grad_weights;
  a.unique_rows = unique_rows;
  a.num_unique = num_unique;
  a.keys_in = (K *)(ws + L.keys_in);
  a.keys = (K *)(ws + L.keys);
  a.pos_in = (uint32_t *)(ws + L.pos_in);
  a.pos = (uint32_t *)(ws + L.pos);
  a.chunk_heads = (uint32_t *)(ws + L.chunk_heads);
  a.block_heads = (uint32_t *)(ws + L.block_heads);
  a.state = (uint32_t *)(ws + L.state);
  a.part = (float *)(ws + L.part);
  a.sentinel = (K)desc->total_rows;
  a.n = n;
  a.F = desc->num_tables;
  a.D = desc->dim;
  a.token = desc->layout == HSTU_EMB_TOKEN;
  a.per_table = a.token ? n / a.F : 0;
  a.nchunks = (int)((n + CHUNK - 1) / CHUNK);
  a.nblocks = (int)((n + HEAD_BLOCK - 1) / HEAD_BLOCK);
  a.scanned = a.nblocks > HEAD_SUM_BLOCKS;
  const int cpr = a.D / elt_n(desc);
  const int cpb = chunk_cpb(cpr);
  a.ngroups = (a.nchunks + cpb - 1) / cpb;
  hipError_t e;
  prof::Scope ps("emb_bwd", s);
  hipLaunchKernelGGL(emb_keys_kernel<K>, dim3((unsigned)((n + ET - 1) / ET)), dim3(ET), 0, s, a);
  if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "embedding key launch");
  size_t tb = L.tmp_bytes;
  e = rocprim::radix_sort_pairs<SortConfig>(ws + L.tmp, tb, a.keys_in, a.keys, a.pos_in, a.pos,
                                (unsigned)n, 0, key_bits(desc->total_rows), s);
  if (e != hipSuccess) return hip_fail(e, "embedding key sort");
  hipLaunchKernelGGL(emb_heads_kernel<K>, dim3((unsigned)a.nblocks), dim3(ET), 0, s, a);
  if (a.scanned) hipLaunchKernelGGL(emb_scan_kernel<K>, dim3(1), dim3(1024), 0, s, a);
  if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "embedding head launch");
  const unsigned grid_c = (unsigned)a.ngroups, grid_f = grid_c;
  if (desc->dtype == HSTU_F32) {
    hipLaunchKernelGGL((emb_chunk_kernel<float, K>), dim3(grid_c), dim3(ET), 0, s, a);
    hipLaunchKernelGGL((emb_fixup_kernel<float, K>), dim3(grid_f), dim3(ET), 0, s, a);
  } else {
    hipLaunchKernelGGL((emb_chunk_kernel<u16, K>), dim3(grid_c), dim3(ET), 0, s, a);
    hipLaunchKernelGGL((emb_fixup_kernel<u16, K>), dim3(grid_f), dim3(ET), 0, s, a);
  }
  if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "embedding chunk launch");
  return HSTU_OK;
}

}  // namespace
}  // namespace hstu

using namespace hstu;

extern "C" int hstu_jagged_embedding_fwd(const hstu_emb_desc *desc, const void *weights,
                                         const int64_t *ids, void *out, void *stream) {
  clear_last_error();
  int rc = check_desc(desc);
  if (rc) return rc;
  if (desc->num_ids == 0) return HSTU_OK;
  if (!weights || !ids || !out) return fail(HSTU_EINVAL, "weights, ids and out must be non-null");
  const hipStream_t s = (hipStream_t)stream;
  FwdArgs a{};
  a.w = weights;
  a.ro = desc->row_offsets;
  a.io = desc->id_offsets;
  a.ids = ids;
  a.out = out;
  a.n = desc->num_ids;
  a.F = desc->num_tables;
  a.D = desc->dim;
  a.token = desc->layout == HSTU_EMB_TOKEN;
  a.per_table = a.token ? a.n / a.F : 0;
  a.total_rows = desc->total_rows;
  const int cpr = a.D / elt_n(desc);
  a.rows_per_block = std::max(1, ET * FWD_UNROLL / cpr);
  if (a.rows_per_block == 1 && cpr > ET * FWD_UNROLL)
    return fail(HSTU_ENOTSUP, "dim %d: a row exceeds one work-group's chunks", a.D);
  const int64_t grid = (a.n + a.rows_per_block - 1) / a.rows_per_block;
  {
    prof::Scope ps("emb_fwd", s);
    if (desc->dtype == HSTU_F32)
      hipLaunchKernelGGL(emb_fwd_kernel<float>, dim3((unsigned)grid), dim3(ET), 0, s, a);
    else
      hipLaunchKernelGGL(emb_fwd_kernel<u16>, dim3((unsigned)grid), dim3(ET), 0, s, a);
  }
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? HSTU_OK : hip_fail(e, "embedding forward launch");
}

extern "C" size_t hstu_jagged_embedding_bwd_workspace_bytes(const hstu_emb_desc *desc) {
  clear_last_error();
  if (check_desc(desc)) return 0;
  size_t tmp = 0;
  const hipError_t e = lib_tmp_bytes(desc, &tmp);
  if (e != hipSuccess) {
    hip_fail(e, "sort workspace query");
    return 0;
  }
  return bwd_layout(desc, tmp).total;
}

extern "C" int hstu_jagged_embedding_bwd(const hstu_emb_desc *desc, const int64_t *ids,
                                         const void *dout, float *grad_weights,
                                         int64_t *unique_rows, int32_t *num_unique,
                                         void *workspace, size_t workspace_bytes,
                                         void *stream) {
  clear_last_error();
  int rc = check_desc(desc);
  if (rc) return rc;
  const hipStream_t s = (hipStream_t)stream;
  const int64_t n = desc->num_ids;
  if (n == 0) {
    if (num_unique) {
      hipLaunchKernelGGL(emb_count_zero_kernel, dim3(1), dim3(1), 0, s, num_unique);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return hip_fail(e, "embedding backward launch");
    }
    return HSTU_OK;
  }
  if (!ids || !dout || !grad_weights)
    return fail(HSTU_EINVAL, "ids, dout and grad_weights must be non-null");
  size_t tmp = 0;
  hipError_t e = lib_tmp_bytes(desc, &tmp);
  if (e != hipSuccess) return hip_fail(e, "sort workspace query");
  const BwdLayout L = bwd_layout(desc, tmp);
  rc = check_workspace_bytes(L.total, workspace, workspace_bytes);
  if (rc) return rc;
  return small_keys(desc)
             ? bwd_launch<uint32_t>(desc, ids, dout, grad_weights, unique_rows, num_unique,
                                    (char *)workspace, L, s)
             : bwd_launch<uint64_t>(desc, ids, dout, grad_weights, unique_rows, num_unique,
                                    (char *)workspace, L, s);
}
