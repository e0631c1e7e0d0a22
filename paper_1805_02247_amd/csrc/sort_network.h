// Wavefront sorting network and run detection of the cell sort (sort.hip), also used by the
// kernels that count segments as they write the keys (cic.hip). Include inside namespace pmr's
// anonymous namespace.
#pragma once

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

// ---------------------------------------------------------------- wavefront sorting network
// Ascending bitonic sort of 64 K values, element e * 64 + lane in v[e], by lane moves on the
// vector units. The kernels that use it are bound by its instructions, so each compare and
// exchange is written to need as few as possible (two at most distances):
//   * the element a lane keeps, the smaller or the larger of its own and its partner's, is
//     the median of the two and a bound (0 or ~0) that is constant per lane and distance;
//   * the first stage of a level up to 16 compares with the mirrored lane (i ^ (k - 1)), which
//     leaves both halves ascending, so no stage needs a direction;
//   * larger levels take their descending halves as complemented values sorted ascending;
//   * lane ^ 1, ^ 2, ^ 3 are quad permutations, ^ 7 and ^ 15 the mirrors of half rows and rows,
//     ^ 8 the rotation of a row by 8, ^ 4 two moves (^ 7, ^ 3); for ^ 16 and ^ 32 the gfx950 row
//     swap of two copies of the value leaves own and partner's value in the pair, in either
//     order, which is all the median needs.
__device__ __forceinline__ uint32_t med3(uint32_t x, uint32_t y, uint32_t z) {
  const uint32_t lo = x < y ? x : y, hi = x < y ? y : x;
  const uint32_t m = hi < z ? hi : z;
  return lo < m ? m : lo;
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_mov(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}

// Bound of the compare and exchange whose upper elements are the lanes with bit J set.
template <int J>
__device__ __forceinline__ uint32_t bound() {
  return (lane_id() & J) ? ~0u : 0u;
}

// Compare and exchange with lane ^ X; the lanes with bit UP set keep the larger value.
template <int X, int UP>
__device__ __forceinline__ uint32_t exchange(uint32_t v) {
  if constexpr (X == 16) {
    const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return med3(p[0], p[1], bound<UP>());
  } else if constexpr (X == 32) {
    const auto p = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return med3(p[0], p[1], bound<UP>());
  } else {
    uint32_t o;
    if constexpr (X == 1) o = dpp_mov<0xB1>(v);
    if constexpr (X == 2) o = dpp_mov<0x4E>(v);
    if constexpr (X == 3) o = dpp_mov<0x1B>(v);
    if constexpr (X == 4) o = dpp_mov<0x1B>(dpp_mov<0x141>(v));
    if constexpr (X == 7) o = dpp_mov<0x141>(v);
    if constexpr (X == 8) o = dpp_mov<0x128>(v);
    if constexpr (X == 15) o = dpp_mov<0x140>(v);
    return med3(v, o, bound<UP>());
  }
}

template <int X, int UP, int K>
__device__ __forceinline__ void exchange_all(uint32_t (&v)[K]) {
#pragma unroll
  for (int e = 0; e < K; ++e) v[e] = exchange<X, UP>(v[e]);
}

// Half-cleaners of distances J, J / 2, ..., 1 across the lanes.
template <int J, int K>
__device__ __forceinline__ void clean(uint32_t (&v)[K]) {
  exchange_all<J, J>(v);
  if constexpr (J > 1) clean<J / 2>(v);
}

// Each of K independent registers ascending across its 64 lanes (together, so that one's lane
// moves fill the wait states of the other's).
template <int K>
__device__ __forceinline__ void wave_sort_each(uint32_t (&v)[K]) {
  const uint32_t b16 = bound<16>(), b32 = bound<32>();
  // descending runs as complements: of 16 (bit 4) and of 32 (bit 5)
#pragma unroll
  for (int e = 0; e < K; ++e) v[e] ^= b16 ^ b32;
  exchange_all<1, 1>(v);
  exchange_all<3, 2>(v);
  clean<1>(v);
  exchange_all<7, 4>(v);
  clean<2>(v);
  exchange_all<15, 8>(v);
  clean<4>(v);
#pragma unroll
  for (int e = 0; e < K; ++e) v[e] ^= b16;
  clean<16>(v);
#pragma unroll
  for (int e = 0; e < K; ++e) v[e] ^= b32;
  clean<32>(v);
}

// The 64 K values of K registers ascending, element e * 64 + lane in v[e].
template <int K>
__device__ __forceinline__ void wave_sort(uint32_t (&v)[K]) {
  static_assert(K == 1 || K == 2 || K == 4, "64, 128 or 256 values");
  // descending runs as complements: of 64 (odd e) and of 128 (e & 2); e = 3 is both
  if constexpr (K >= 2) v[1] = ~v[1];
  if constexpr (K == 4) v[2] = ~v[2];
  wave_sort_each<K>(v);
  if constexpr (K >= 2) {
#pragma unroll
    for (int e = 1; e < K; e += 2) v[e] = ~v[e];
#pragma unroll
    for (int e = 0; e < K; e += 2) {
      const uint32_t x = v[e], y = v[e + 1];
      v[e] = x < y ? x : y;
      v[e + 1] = x < y ? y : x;
    }
    clean<32>(v);
  }
  if constexpr (K == 4) {
#pragma unroll
    for (int e = 2; e < 4; ++e) v[e] = ~v[e];
#pragma unroll
    for (int d = 2; d >= 1; --d)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if ((e & d) == 0) {
          const uint32_t x = v[e], y = v[e + d];
          v[e] = x < y ? x : y;
          v[e + d] = x < y ? y : x;
        }
    clean<32>(v);
  }
}

// The 64 (row, lane) pairs of a wavefront sorted by a bitonic network across lanes, so that
// equal rows form runs: the first lane of each run then issues one atomic for the whole run,
// all runs at once (instead of one round trip per distinct row). Rows must be <= 2^25 (the
// caller checks), so that no entry equals the end marker ~0 that lanes past the end carry.
// Runs of equal rows among the sorted (row << 6 | lane) values: for each lane the row, the
// first lane of its run and the run's length (valid only for real entries).
struct WaveRuns {
  uint32_t row;
  int head, len;
  bool ok;
};

__device__ __forceinline__ WaveRuns wave_runs(uint32_t sorted) {
  const int lane = lane_id();
  WaveRuns w;
  w.ok = sorted != ~0u;
  w.row = sorted >> 6;
  const uint32_t prev = __shfl_up(w.row, 1, 64);
  const bool head = w.ok && (lane == 0 || prev != w.row);
  const uint64_t heads = __ballot(head);
  const uint64_t valid = __ballot(w.ok);
  const uint64_t upto = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);  // lanes 0..lane
  w.head = 63 - __clzll((long long)(heads & upto));
  const uint64_t after = heads & ~upto;  // heads above this lane
  const int end = after ? __ffsll((unsigned long long)after) - 1 : __popcll(valid);
  w.len = end - w.head;
  return w;
}

// Adds one per lane to the counters of the lanes' segments (all 64 lanes active): one atomic per
// run of equal segments in the wavefront.
__device__ __forceinline__ void count_segments(uint32_t* __restrict__ cnt, uint32_t segment) {
  const int lane = lane_id();
  uint32_t v[1] = {(segment << 6) | (uint32_t)lane};
  wave_sort_each<1>(v);
  const WaveRuns w = wave_runs(v[0]);
  if (w.head == lane) atomicAdd(&cnt[w.row], (uint32_t)w.len);
}
