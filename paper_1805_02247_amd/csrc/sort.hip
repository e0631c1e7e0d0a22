// The cell sort of the particles: the unique (cell key, id) order, the row index of the
// sorted stream and the payloads that travel with it, in four steps.
//
//   1. counts:     particles per row segment (item, ix, iy and the top bits of iz: a row or
//                  a part of it, cell_sort_split) = key >> (log2(nm) - split), with one
//                  atomic per distinct segment per wavefront, taken by the kernel that writes the
//                  keys (sort_count) on counters that each row sort leaves at zero.
//   2. scan:       exclusive scan of the counts -> row_start (the row index the paints and
//                  gathers use) and a cursor per segment.
//   3. bucket:     every particle into its segment's range, at a slot taken from the segment's
//                  cursor (the order inside a segment depends on the timing of the atomics),
//                  as its composite (iz within the segment, id) in one word.
//   4. row sort:   each segment's composites sorted; they are unique per particle, so the
//                  result is the (key, id) order whatever the bucket order was. One launch: a
//                  wavefront sorts segments of up to 256 entries in registers (bitonic network
//                  across lanes), the first workgroups of the grid those of up to 4096 in LDS,
//                  or larger ones (which only occur in very dense layouts) with a stable LSD
//                  radix sort in global memory. Every sorted entry is written with its
//                  payload (gathered by id) and its inverse permutation entry.
//
// Compulsory traffic: the id-order keys read once (bucket), one word written and read
// per particle in the buckets, the sorted keys, ids and payload written; no pass over
// 8-bit digits of the whole key array.
#include "pmr_internal.h"

namespace pmr {
namespace {

constexpr int TB = 256;
constexpr int WAVE_ROW_MAX = 256;    // tier 1: one wavefront, 4 entries per lane
constexpr int BLOCK_ROW_MAX = 4096;  // tier 2: one workgroup, 16 entries per thread in LDS
constexpr size_t LONG_BLOCKS = 1024;  // workgroups that take the rows beyond tier 1
constexpr int SCAN_ITEMS = 16;
constexpr int SCAN_TILE = TB * SCAN_ITEMS;  // counts per scan block
constexpr int SCAN1_TB = 1024;              // threads of the one-launch scan
constexpr int SCAN1_MAX_BLOCKS = 64;        // scan blocks up to which it is used

#include "sort_network.h"

__device__ __forceinline__ uint64_t lanes_below() {
  const int l = lane_id();
  return l == 0 ? 0ull : (~0ull >> (64 - l));
}

__global__ void fill_u32_kernel(uint32_t* __restrict__ p, size_t n, uint32_t v) {
  for (size_t i = (size_t)blockIdx.x * TB + threadIdx.x; i < n; i += (size_t)gridDim.x * TB)
    p[i] = v;
}

// ---------------------------------------------------------------- 1. counts
// Particles are visited in `order` (a permutation of the ids, nullable: id order). The
// previous step's sorted order groups particles by their old cell, and a particle moves
// about a cell per step, so a wavefront of it falls in one or two new rows.
__device__ __forceinline__ uint32_t visit(const uint32_t* __restrict__ order, int g) {
  return order ? order[g] : (uint32_t)g;
}

// Groups of 64 particles per wavefront and launch (each thread holds one particle of each
// group, loaded together so that the loads of the groups overlap). Two measured 1.5% faster
// for the sort than four at 256^3 on 512^3 and the same at 128^3 x 4; eight was slower.
constexpr int GROUPS = 2;

__device__ __forceinline__ int group_base(int q) {
  return ((blockIdx.x * (TB / 64) + (threadIdx.x >> 6)) * GROUPS + q) * 64;
}

// Counts with one round trip per distinct row (any number of rows); packed row numbers are
// counted by the kernels that write the keys.
__global__ __launch_bounds__(TB) void row_count_loop_kernel(const uint32_t* __restrict__ keys,
                                                            const uint32_t* __restrict__ order,
                                                            int n, int shift,
                                                            uint32_t* __restrict__ cnt) {
  const int g = blockIdx.x * TB + threadIdx.x;
  const bool ok = g < n;
  const uint32_t r = ok ? keys[visit(order, g)] >> shift : 0u;
  uint64_t todo = __ballot(ok);
  while (todo) {
    const int leader = __ffsll((unsigned long long)todo) - 1;
    const uint32_t rl = __shfl(r, leader, 64);
    const uint64_t same = __ballot(ok && r == rl);
    if (lane_id() == leader) atomicAdd(&cnt[rl], (uint32_t)__popcll(same));
    todo &= ~same;
  }
}

// ---------------------------------------------------------------- 2. scan
// Inclusive scan over the block of one value per thread (wavefront shuffles, then the
// wavefront totals); returns the inclusive prefix and the block total.
__device__ __forceinline__ uint32_t block_inclusive_scan(uint32_t v, uint32_t* wsum,
                                                         uint32_t* total) {
  const int lane = lane_id(), w = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) wsum[w] = x;
  __syncthreads();
  uint32_t pre = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < TB / 64; ++i) {
    const uint32_t s = wsum[i];
    if (i < w) pre += s;
    tot += s;
  }
  __syncthreads();
  *total = tot;
  return pre + x;
}

// partial[b] = sum of counts of scan block b
__global__ __launch_bounds__(TB) void scan_reduce_kernel(const uint32_t* __restrict__ cnt,
                                                         size_t rows,
                                                         uint32_t* __restrict__ partial) {
  __shared__ uint32_t wsum[TB / 64];
  const size_t base = (size_t)blockIdx.x * SCAN_TILE + (size_t)threadIdx.x * SCAN_ITEMS;
  uint32_t s = 0;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) s += base + i < rows ? cnt[base + i] : 0u;
  uint32_t tot;
  block_inclusive_scan(s, wsum, &tot);
  if (threadIdx.x == 0) partial[blockIdx.x] = tot;
}

// exclusive scan of the block partials in place (one workgroup, any number of blocks)
__global__ __launch_bounds__(TB) void scan_partials_kernel(uint32_t* __restrict__ partial,
                                                           int nb) {
  __shared__ uint32_t wsum[TB / 64];
  uint32_t carry = 0;
  for (int b0 = 0; b0 < nb; b0 += TB) {
    const int b = b0 + threadIdx.x;
    const uint32_t v = b < nb ? partial[b] : 0u;
    uint32_t tot;
    const uint32_t inc = block_inclusive_scan(v, wsum, &tot);
    if (b < nb) partial[b] = carry + inc - v;
    carry += tot;
  }
}

// start[r] = exclusive prefix of the counts of the segments; cursor[r] = start[r];
// start[rows] = n (the total); the row index of the caller gets the start of every
// (1 << split)-th segment (the first segment of each row).
__global__ __launch_bounds__(TB) void scan_write_kernel(const uint32_t* __restrict__ cnt,
                                                        size_t rows,
                                                        const uint32_t* __restrict__ partial,
                                                        uint32_t n,
                                                        uint32_t* __restrict__ row_start,
                                                        uint32_t* __restrict__ cursor,
                                                        uint32_t* __restrict__ seg_start,
                                                        int split) {
  __shared__ uint32_t wsum[TB / 64];
  const size_t base = (size_t)blockIdx.x * SCAN_TILE + (size_t)threadIdx.x * SCAN_ITEMS;
  uint32_t v[SCAN_ITEMS];
  uint32_t s = 0;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    v[i] = base + i < rows ? cnt[base + i] : 0u;
    s += v[i];
  }
  uint32_t tot;
  uint32_t run = partial[blockIdx.x] + block_inclusive_scan(s, wsum, &tot) - s;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    const size_t r = base + i;
    if (r < rows) {
      seg_start[r] = run;
      cursor[r] = run;
      if ((r & (((size_t)1 << split) - 1)) == 0) row_start[r >> split] = run;
    }
    run += v[i];
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    seg_start[rows] = n;
    row_start[rows >> split] = n;
  }
}

// The whole scan in one launch, for up to SCAN1_MAX_BLOCKS tiles: a workgroup sums every count
// before its tile (at most 1 MB, from L2) instead of waiting for two more launches to reduce
// and scan the tiles' totals.
__global__ __launch_bounds__(SCAN1_TB) void scan_one_kernel(const uint32_t* __restrict__ cnt,
                                                            size_t rows, uint32_t n,
                                                            uint32_t* __restrict__ row_start,
                                                            uint32_t* __restrict__ cursor,
                                                            uint32_t* __restrict__ seg_start,
                                                            int split) {
  constexpr int WAVES = SCAN1_TB / 64;
  static_assert(SCAN_TILE == 4 * SCAN1_TB, "four counts per thread");
  __shared__ uint32_t wsum[2][WAVES];
  const int t = threadIdx.x, lane = lane_id(), w = t >> 6;
  const uint4* c4 = reinterpret_cast<const uint4*>(cnt);  // rows is a multiple of 4
  const size_t tile = (size_t)blockIdx.x * SCAN1_TB + t;  // this thread's four counts
  uint32_t before = 0;
#pragma unroll 8
  for (int b = 0; b < (int)blockIdx.x; ++b) {
    const uint4 c = c4[(size_t)b * SCAN1_TB + t];
    before += c.x + c.y + c.z + c.w;
  }
  uint4 v = make_uint4(0u, 0u, 0u, 0u);
  if (4 * tile < rows) v = c4[tile];
  const uint32_t own = v.x + v.y + v.z + v.w;
  uint32_t x = own;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
    before += __shfl_xor(before, d, 64);
  }
  if (lane == 63) {
    wsum[0][w] = x;
    wsum[1][w] = before;
  }
  __syncthreads();
  uint32_t run = x - own;
#pragma unroll
  for (int i = 0; i < WAVES; ++i) run += (i < w ? wsum[0][i] : 0u) + wsum[1][i];
  if (4 * tile < rows) {
    const uint4 o = make_uint4(run, run + v.x, run + v.x + v.y, run + v.x + v.y + v.z);
    reinterpret_cast<uint4*>(cursor)[tile] = o;
    reinterpret_cast<uint4*>(seg_start)[tile] = o;
    const uint32_t e[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const size_t r = 4 * tile + i;
      if ((r & (((size_t)1 << split) - 1)) == 0) row_start[r >> split] = e[i];
    }
  }
  if (blockIdx.x == 0 && t == 0) {
    seg_start[rows] = n;
    row_start[rows >> split] = n;
  }
}

// ---------------------------------------------------------------- 3. buckets
// One word per particle: its cell within the segment above its id, which the row sort can
// order without another look at the keys (the gather of the keys by id was its second
// dependent load).
__device__ __forceinline__ uint32_t composite(uint32_t key, uint32_t zmask, int idbits,
                                              uint32_t id) {
  return ((key & zmask) << idbits) | id;
}

__global__ __launch_bounds__(TB) void bucket_kernel(const uint32_t* __restrict__ keys,
                                                    const uint32_t* __restrict__ order, int n,
                                                    int shift, int idbits,
                                                    uint32_t* __restrict__ cursor,
                                                    uint32_t* __restrict__ bucket) {
  const int lane = lane_id();
  const uint32_t zmask = (1u << shift) - 1u;
  uint32_t id[GROUPS], v[GROUPS];
#pragma unroll
  for (int q = 0; q < GROUPS; ++q) {
    const int g = group_base(q) + lane;
    id[q] = g < n ? visit(order, g) : 0u;
  }
#pragma unroll
  for (int q = 0; q < GROUPS; ++q) {
    const int g = group_base(q) + lane;
    const uint32_t key = g < n ? keys[id[q]] : 0u;
    v[q] = g < n ? ((key >> shift) << 6) | (uint32_t)lane : ~0u;
    id[q] = composite(key, zmask, idbits, id[q]);
  }
  uint32_t sorted[GROUPS];
#pragma unroll
  for (int q = 0; q < GROUPS; ++q) sorted[q] = v[q];
  wave_sort_each<GROUPS>(sorted);
#pragma unroll
  for (int q = 0; q < GROUPS; ++q) {
    const WaveRuns w = wave_runs(sorted[q]);
    uint32_t base = 0;
    if (w.ok && w.head == lane) base = atomicAdd(&cursor[w.row], (uint32_t)w.len);
    base = __shfl(base, w.ok ? w.head : lane, 64);
    const uint32_t src = __shfl(id[q], (int)(sorted[q] & 63u), 64);
    if (w.ok) bucket[base + (uint32_t)(lane - w.head)] = src;
  }
}

__global__ __launch_bounds__(TB) void bucket_loop_kernel(const uint32_t* __restrict__ keys,
                                                         const uint32_t* __restrict__ order,
                                                         int n, int shift, int idbits,
                                                         uint32_t* __restrict__ cursor,
                                                         uint32_t* __restrict__ bucket) {
  const int g = blockIdx.x * TB + threadIdx.x;
  const bool ok = g < n;
  const uint32_t id = ok ? visit(order, g) : 0u;
  const uint32_t key = ok ? keys[id] : 0u;
  const uint32_t r = key >> shift;
  uint64_t todo = __ballot(ok);
  uint32_t pos = 0;
  while (todo) {
    const int leader = __ffsll((unsigned long long)todo) - 1;
    const uint32_t rl = __shfl(r, leader, 64);
    const bool mine = ok && r == rl;
    const uint64_t same = __ballot(mine);
    uint32_t base = 0;
    if (lane_id() == leader) base = atomicAdd(&cursor[rl], (uint32_t)__popcll(same));
    base = __shfl(base, leader, 64);
    if (mine) pos = base + (uint32_t)__popcll(same & lanes_below());
    todo &= ~same;
  }
  if (ok) bucket[pos] = composite(key, (1u << shift) - 1u, idbits, id);
}

// ---------------------------------------------------------------- 4. row sorts
struct RowSortArgs {
  const uint32_t* row_start;  // [rows + 1]
  const uint32_t* bucket;     // composites (iz << idbits | id) bucketed by row
  uint32_t* keys_sorted;
  uint32_t* ids_sorted;
  const Vec3* pay_in;  // nullable
  Vec3* pay_out;
  uint32_t* inv;       // nullable
  uint32_t* tmp_hi;    // global radix scratch [n] x 2 (rows beyond the LDS tier)
  uint32_t* tmp_lo;
  int shift;
  int idbits;          // bits of the largest id
  size_t rows;
  int long_blocks;     // workgroups at the start of the grid that take the long rows
  int block_rows;      // rows such a workgroup tests per step (<= TB)
  uint32_t* clear;     // counters to clear for the next sort (nullable)
  size_t n_clear;
};

// Writes one sorted entry at sorted position pos of row `row`, with its payload
// (non-temporal: read once, by the paint after the sort) and inverse permutation entry.
// (A separate streaming pass over the sorted ids for these measured no faster at 256^3 on
// 512^3 and 2% slower for the sort at 128^3 x 4: the gather by id costs the same in either.)
__device__ __forceinline__ void emit(const RowSortArgs& a, uint32_t row, uint32_t pos,
                                     uint32_t iz, uint32_t id) {
  a.keys_sorted[pos] = (row << a.shift) | iz;
  a.ids_sorted[pos] = id;
  if (a.pay_out) {
    const Vec3 p = a.pay_in[id];
    __builtin_nontemporal_store(p.x, &a.pay_out[pos].x);
    __builtin_nontemporal_store(p.y, &a.pay_out[pos].y);
    __builtin_nontemporal_store(p.z, &a.pay_out[pos].z);
  }
  if (a.inv) a.inv[id] = pos;
}

__device__ __forceinline__ uint32_t id_of(const RowSortArgs& a, uint32_t v) {
  return v & ((1u << a.idbits) - 1u);
}
__device__ __forceinline__ uint32_t iz_of(const RowSortArgs& a, uint32_t v) {
  return v >> a.idbits;
}

__device__ __forceinline__ void emit_composite(const RowSortArgs& a, uint32_t row, uint32_t pos,
                                               uint32_t v) {
  emit(a, row, pos, iz_of(a, v), id_of(a, v));
}

// Tier 1: each wavefront takes two rows at a time, loading both before sorting either, so
// that their dependent loads (row start, bucket) overlap; rows of 1..256 entries are sorted
// here. (Two rows per step measured 2-3% faster for the sort than one or four, and eight 13%
// slower: more rows in flight cost resident waves.)
constexpr int WAVE_ROWS = 2;

// Rows r0 .. r0 + WAVE_ROWS - 1 by one wavefront.
__device__ __forceinline__ void sort_wave_rows(const RowSortArgs& a, size_t r0) {
  constexpr uint32_t PAD = ~0u;  // sorts after (or ties with) every real entry
  const int lane = lane_id();
  uint32_t start[WAVE_ROWS], cnt[WAVE_ROWS];
#pragma unroll
  for (int q = 0; q < WAVE_ROWS; ++q) {
    const size_t r = r0 + q;
    start[q] = r < a.rows ? a.row_start[r] : 0u;
    cnt[q] = r < a.rows ? a.row_start[r + 1] - start[q] : 0u;
    if (cnt[q] > WAVE_ROW_MAX) cnt[q] = 0;  // the workgroup tiers take it
  }
  uint32_t v[WAVE_ROWS][4];
#pragma unroll
  for (int q = 0; q < WAVE_ROWS; ++q)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t i = e * 64 + lane;
      v[q][e] = i < cnt[q] ? a.bucket[start[q] + i] : PAD;
    }
  if (cnt[0] <= 64 && cnt[1] <= 64) {
    static_assert(WAVE_ROWS == 2, "two rows sorted together");
    uint32_t w[2] = {v[0][0], v[1][0]};
    wave_sort_each<2>(w);
#pragma unroll
    for (int q = 0; q < 2; ++q)
      if (lane < (int)cnt[q]) emit_composite(a, (uint32_t)(r0 + q), start[q] + lane, w[q]);
    return;
  }
#pragma unroll
  for (int q = 0; q < WAVE_ROWS; ++q) {
    if (cnt[q] == 0) continue;
    const uint32_t row = (uint32_t)(r0 + q);
    if (cnt[q] <= 64) {
      uint32_t w1[1] = {v[q][0]};
      wave_sort<1>(w1);
      if (lane < (int)cnt[q]) emit_composite(a, row, start[q] + lane, w1[0]);
    } else if (cnt[q] <= 128) {
      uint32_t w2[2] = {v[q][0], v[q][1]};
      wave_sort<2>(w2);
#pragma unroll
      for (int e = 0; e < 2; ++e)
        if ((uint32_t)(e * 64 + lane) < cnt[q])
          emit_composite(a, row, start[q] + e * 64 + lane, w2[e]);
    } else {
      wave_sort<4>(v[q]);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if ((uint32_t)(e * 64 + lane) < cnt[q])
          emit_composite(a, row, start[q] + e * 64 + lane, v[q][e]);
    }
  }
}

// Stable scatter of one LSD radix pass over 8 bits of the composite held as (hi, lo) pairs,
// src -> dst within one row's range, by one workgroup, chunk by chunk in order.
__device__ void block_radix_pass(const uint32_t* shi, const uint32_t* slo, uint32_t* dhi,
                                 uint32_t* dlo, uint32_t c, int bit, uint32_t* base,
                                 uint32_t (*wcnt)[256]) {
  const int t = threadIdx.x, lane = lane_id(), w = t >> 6;
  auto digit = [&](uint32_t hi, uint32_t lo) -> uint32_t {
    return bit >= 32 ? (hi >> (bit - 32)) & 255u : (lo >> bit) & 255u;
  };
  // histogram -> exclusive digit offsets
  base[t] = 0;
  __syncthreads();
  for (uint32_t i = t; i < c; i += TB) atomicAdd(&base[digit(shi[i], slo[i])], 1u);
  __syncthreads();
  {
    __shared__ uint32_t wsum[TB / 64];
    const uint32_t v = base[t];
    uint32_t tot;
    const uint32_t inc = block_inclusive_scan(v, wsum, &tot);
    base[t] = inc - v;
  }
  __syncthreads();
  for (uint32_t c0 = 0; c0 < c; c0 += TB) {
    const uint32_t i = c0 + t;
    const bool ok = i < c;
    const uint32_t hi = ok ? shi[i] : 0u, lo = ok ? slo[i] : 0u;
    const uint32_t d = ok ? digit(hi, lo) : 0u;
    for (int q = 0; q < TB / 64; ++q) wcnt[q][t] = 0;
    __syncthreads();
    uint64_t m = __ballot(ok);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bool on = (d >> b) & 1u;
      const uint64_t bal = __ballot(on);
      m &= on ? bal : ~bal;
    }
    const uint32_t rank = (uint32_t)__popcll(m & lanes_below());
    if (ok && rank == 0) wcnt[w][d] = (uint32_t)__popcll(m);
    __syncthreads();
    if (ok) {
      uint32_t pos = base[d] + rank;
      for (int q = 0; q < w; ++q) pos += wcnt[q][d];
      dhi[pos] = hi;
      dlo[pos] = lo;
    }
    __syncthreads();
    uint32_t add = 0;
    for (int q = 0; q < TB / 64; ++q) add += wcnt[q][t];
    base[t] += add;
    __syncthreads();
  }
}

// Tier 2 (rows of 257..4096 entries: bitonic sort in LDS) and tier 3 (larger rows: stable
// LSD radix passes in global memory over the digits that vary in the row). A workgroup
// tests the lengths of block_rows rows together and then sorts the long ones one after the
// other (rows are independent, so the order in which they are done does not matter). In a
// clustered field the long rows are neighbours and a workgroup that tests neighbours sorts them
// all in a row, so the rows of a workgroup come from places far apart, RUN consecutive ones from
// each. 128^3 particles in a cluster (sigma a tenth of the box) per sort: 823 us with
// neighbours, 490 with runs of 16, 465 with 8 on 256^3, 1130, 848 and 663 on 128^3; tighter (a
// fiftieth) 3480, 2590 and 2210. An even field has no long rows: 270 and 271.
constexpr int RUN = 8;
__device__ __forceinline__ void sort_long_rows(const RowSortArgs& a, uint32_t* s, uint32_t* found,
                                               int* nfound) {
  __shared__ uint32_t red[2][TB / 64];
  uint32_t* base = s;  // tier 3 has no use for the LDS tile itself
  uint32_t(*wcnt)[256] = reinterpret_cast<uint32_t(*)[256]>(s + 256);
  const int t = threadIdx.x;
  const uint32_t rows = (uint32_t)a.rows;  // at most 2^31 segments
  const uint32_t apart = (uint32_t)a.long_blocks * RUN;
  for (uint32_t r0 = blockIdx.x * RUN; r0 < rows; r0 += (uint32_t)a.long_blocks * a.block_rows) {
    if (t == 0) *nfound = 0;
    __syncthreads();
    const uint32_t mine = r0 + (uint32_t)t / RUN * apart + (uint32_t)t % RUN;
    if (t < a.block_rows && mine < rows &&
        a.row_start[mine + 1] - a.row_start[mine] > WAVE_ROW_MAX)
      found[atomicAdd(nfound, 1)] = mine;
    __syncthreads();
    const int nf = *nfound;
    for (int f = 0; f < nf; ++f) {
      const uint32_t r = found[f];
      const uint32_t start = a.row_start[r];
      const uint32_t c = a.row_start[r + 1] - start;
      const uint32_t row = r;
      if (c <= BLOCK_ROW_MAX) {
        uint32_t p2 = 512;
        while (p2 < c) p2 <<= 1;
        for (uint32_t i = t; i < p2; i += TB) s[i] = i < c ? a.bucket[start + i] : ~0u;
        __syncthreads();
        for (uint32_t k = 2; k <= p2; k <<= 1) {
          for (uint32_t j = k >> 1; j > 0; j >>= 1) {
            for (uint32_t q = t; q < p2 / 2; q += TB) {
              const uint32_t i = ((q & ~(j - 1)) << 1) | (q & (j - 1));
              const uint32_t p = i | j;
              const bool up = (i & k) == 0;
              const uint32_t x = s[i], y = s[p];
              if ((x > y) == up) {
                s[i] = y;
                s[p] = x;
              }
            }
            __syncthreads();
          }
        }
        for (uint32_t i = t; i < c; i += TB) emit_composite(a, row, start + i, s[i]);
        __syncthreads();
        continue;
      }
      // tier 3: (hi, lo) = (iz, id) pairs; A = the row's range of the sorted outputs, B = the
      // radix scratch
      uint32_t* ahi = a.keys_sorted + start;
      uint32_t* alo = a.ids_sorted + start;
      uint32_t* bhi = a.tmp_hi + start;
      uint32_t* blo = a.tmp_lo + start;
      uint32_t orv[2] = {0u, 0u}, andv[2] = {~0u, ~0u};
      for (uint32_t i = t; i < c; i += TB) {
        const uint32_t v = a.bucket[start + i];
        const uint32_t hi = iz_of(a, v), id = id_of(a, v);
        ahi[i] = hi;
        alo[i] = id;
        orv[0] |= hi;
        andv[0] &= hi;
        orv[1] |= id;
        andv[1] &= id;
      }
      // bits that vary across the row (passes over constant digits are skipped)
      uint32_t var[2];
      for (int h = 0; h < 2; ++h) {
        uint32_t o = orv[h], n = andv[h];
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
          o |= __shfl_xor(o, d, 64);
          n &= __shfl_xor(n, d, 64);
        }
        if (lane_id() == 0) {
          red[0][t >> 6] = o;
          red[1][t >> 6] = n;
        }
        __syncthreads();
        o = 0u;
        n = ~0u;
        for (int q = 0; q < TB / 64; ++q) {
          o |= red[0][q];
          n &= red[1][q];
        }
        var[h] = o ^ n;
        __syncthreads();
      }
      bool in_a = true;
      for (int bit = 0; bit < 64; bit += 8) {
        const uint32_t vm = bit >= 32 ? var[0] >> (bit - 32) : var[1] >> bit;
        if ((vm & 255u) == 0) continue;
        __syncthreads();  // the previous pass's writes
        if (in_a)
          block_radix_pass(ahi, alo, bhi, blo, c, bit, base, wcnt);
        else
          block_radix_pass(bhi, blo, ahi, alo, c, bit, base, wcnt);
        in_a = !in_a;
      }
      __syncthreads();
      const uint32_t* fhi = in_a ? ahi : bhi;
      const uint32_t* flo = in_a ? alo : blo;
      // each thread reads and rewrites only its own indices of A (in place when the last pass
      // landed there)
      for (uint32_t i = t; i < c; i += TB) emit(a, row, start + i, fhi[i], flo[i]);
      __syncthreads();
    }
    __syncthreads();  // every thread has read nfound before it is reset
  }
}

// Both tiers in one launch: the long rows' workgroups come first in the grid, so that their
// longer work runs beside the wavefront tier instead of after it (as a launch of its own it
// cost 10-24 us per sort), and the wavefront tier's blocks are mapped so that neighbouring
// rows, whose payload lines overlap, share an L2.
__global__ __launch_bounds__(TB) void row_sort_kernel(RowSortArgs a) {
  __shared__ uint32_t s[BLOCK_ROW_MAX];
  __shared__ uint32_t found[TB];
  __shared__ int nfound;
  if (a.clear)
    for (size_t i = (size_t)blockIdx.x * TB + threadIdx.x; i < a.n_clear;
         i += (size_t)gridDim.x * TB)
      a.clear[i] = 0u;
  if ((int)blockIdx.x < a.long_blocks) {
    sort_long_rows(a, s, found, &nfound);
    return;
  }
  const int b = xcd_block(blockIdx.x - a.long_blocks, gridDim.x - a.long_blocks);
  sort_wave_rows(a, ((size_t)b * (TB / 64) + (threadIdx.x >> 6)) * WAVE_ROWS);
}

int grid_for(size_t n, int per_block) {
  const size_t b = (n + per_block - 1) / per_block;
  return (int)(b < 1 ? 1 : b);
}

}  // namespace

// Row segments: the sort works on segments of 2^split cells of a row (split low bits of iz
// moved into the segment number), chosen so that the (iz, id) composite of a segment fits
// 32 bits and a segment holds 64 particles or fewer on average (so the wavefront tier
// takes nearly every segment).
int cell_sort_split(int n, size_t rows, int shift) {
  int idbits = 0;
  while (idbits < 32 && ((size_t)1 << idbits) < (size_t)n) ++idbits;
  int split = shift + idbits > 32 ? shift + idbits - 32 : 0;
  while (split < shift && (double)n / (double)(rows << split) > 64.0) ++split;
  return split > shift ? shift : split;
}

size_t cell_sort_scratch_bytes(int n, size_t rows, int shift) {
  const size_t segs = rows << cell_sort_split(n, rows, shift);
  const size_t nb = (segs + SCAN_TILE - 1) / SCAN_TILE;
  // cursors, segment starts, scan partials, buckets, radix scratch (hi, lo)
  return (2 * segs + 1 + nb + 64 + 3 * (size_t)n) * sizeof(uint32_t) + 4 * 256;
}

size_t cell_sort_segments(int n, size_t rows, int shift) {
  return rows << cell_sort_split(n, rows, shift);
}

bool cell_sort_packed(int n, size_t rows, int shift) {
  return cell_sort_segments(n, rows, shift) <= ((size_t)1 << 25);
}

SortCount sort_count(uint32_t* cnt, int n, size_t rows, int shift) {
  return SortCount{cnt, shift - cell_sort_split(n, rows, shift)};
}

void launch_sort_clear(uint32_t* cnt, size_t n, hipStream_t s) {
  const size_t b = (n + TB * 8 - 1) / (TB * 8);
  fill_u32_kernel<<<(int)(b < 1 ? 1 : b > 1024 ? 1024 : b), TB, 0, s>>>(cnt, n, 0u);
}

void launch_cell_sort(const uint32_t* keys, const uint32_t* order, int n, int shift,
                      size_t rows, uint32_t* keys_sorted, uint32_t* ids_sorted,
                      uint32_t* row_start, uint32_t* cnt, bool counted, size_t n_clear,
                      void* scratch, const Vec3* pay_in, Vec3* pay_out, uint32_t* inv,
                      hipStream_t s) {
  const int split = cell_sort_split(n, rows, shift);
  const int sshift = shift - split;  // key >> sshift = segment
  const size_t segs = rows << split;
  const size_t nb = (segs + SCAN_TILE - 1) / SCAN_TILE;
  uint32_t* cursor = (uint32_t*)scratch;
  uint32_t* seg_start = cursor + segs;
  uint32_t* partial = seg_start + segs + 4;
  uint32_t* bucket = partial + nb + 64;
  uint32_t* tmp_hi = bucket + n;
  uint32_t* tmp_lo = tmp_hi + n;
  int idbits = 0;
  while (((size_t)1 << idbits) < (size_t)n) ++idbits;  // at most 31: n is an int
  // (segment << 6 | lane) fits 32 bits below the end marker ~0 for the wavefront sort of
  // the segment numbers
  const bool packed = cell_sort_packed(n, rows, shift);
  if (!counted)
    row_count_loop_kernel<<<grid_for(n, TB), TB, 0, s>>>(keys, order, n, sshift, cnt);
  // The one-launch scan reads every count before a tile, so its last workgroup's share grows
  // with the tiles, while three launches cost ~18-20 us up to there: 5.3 us at 8 tiles (128^3
  // particles), 9.2 at 32 (4 items of them), 14 at 64 (512^2 segments). It needs the counts on
  // 16 bytes.
  if (nb <= SCAN1_MAX_BLOCKS && (((uintptr_t)scratch | (uintptr_t)cnt) & 15) == 0) {
    scan_one_kernel<<<(int)nb, SCAN1_TB, 0, s>>>(cnt, segs, (uint32_t)n, row_start, cursor,
                                                 seg_start, split);
  } else {
    scan_reduce_kernel<<<(int)nb, TB, 0, s>>>(cnt, segs, partial);
    scan_partials_kernel<<<1, TB, 0, s>>>(partial, (int)nb);
    scan_write_kernel<<<(int)nb, TB, 0, s>>>(cnt, segs, partial, (uint32_t)n, row_start, cursor,
                                              seg_start, split);
  }
  if (packed)
    bucket_kernel<<<grid_for(n, TB * GROUPS), TB, 0, s>>>(keys, order, n, sshift, idbits, cursor,
                                                          bucket);
  else
    bucket_loop_kernel<<<grid_for(n, TB), TB, 0, s>>>(keys, order, n, sshift, idbits, cursor,
                                                      bucket);
  RowSortArgs a{};
  a.row_start = seg_start;
  a.bucket = bucket;
  a.keys_sorted = keys_sorted;
  a.ids_sorted = ids_sorted;
  a.pay_in = pay_in;
  a.pay_out = pay_out;
  a.inv = inv;
  a.tmp_hi = tmp_hi;
  a.tmp_lo = tmp_lo;
  a.shift = sshift;
  a.idbits = idbits;
  a.rows = segs;
  a.clear = n_clear ? cnt : nullptr;
  a.n_clear = n_clear;
  // rows tested per workgroup step of the long tier: TB, halved (down to 32) while that leaves
  // workgroups of it without rows, so that the long rows spread over the chip
  a.block_rows = TB;
  while (a.block_rows > 32 && segs / (size_t)a.block_rows < LONG_BLOCKS) a.block_rows /= 2;
  const size_t chunks = (segs + a.block_rows - 1) / a.block_rows;
  a.long_blocks = chunks < LONG_BLOCKS ? (int)chunks : (int)LONG_BLOCKS;
  // one wavefront per WAVE_ROWS segments
  const size_t need = (segs + WAVE_ROWS * (TB / 64) - 1) / (WAVE_ROWS * (TB / 64));
  row_sort_kernel<<<a.long_blocks + (int)need, TB, 0, s>>>(a);
}

}  // namespace pmr
