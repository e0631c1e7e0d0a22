// CIC paint building blocks shared by the paint kernels (cic.hip) and the paint fused with
// the first FFT pass (fft_kernels.h): sorted-stream chunks, the wave-level segmented scan and
// the phase-ordered deposit into a wavefront's LDS rows. Include inside namespace pmr's
// anonymous namespace.
#pragma once


// Segmented inclusive scan over the 64 lanes by equal key, on DPP lane moves (VALU, no
// LDS): row_shr 1, 2, 4, 8 inside each row of 16 lanes, then row_bcast 15 and row_bcast 31
// across rows. Keys are sorted across the lanes, so "source key == my key" means the
// source lane is in my segment. A key whose DPP source is out of range or in a row the
// move leaves out reads ~0 (at most the key of the very last cell, whose added value is
// then 0); the in-row shifts read values with the bound control (out of range reads 0)
// and no old operand, so no register has to be cleared before them, and the row
// broadcasts, which leave rows out, read 0 there from a cleared old operand. The
// neighbour keys (previous and next lane across the whole wavefront) come from the DPP
// wavefront shifts, VALU moves with no LDS round trip; lanes 0 and 63, which have no
// neighbour there, are handled by the lane tests that follow.
template <int CTRL, int RMASK>
__device__ __forceinline__ float dpp_f(float src) {
  if constexpr (RMASK == 0xF)  // every row written: out-of-range lanes read 0
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(src), CTRL, RMASK, 0xF, true));
  else  // rows left out keep the old operand: 0
    return __int_as_float(
        __builtin_amdgcn_update_dpp(0, __float_as_int(src), CTRL, RMASK, 0xF, false));
}
template <int CTRL, int RMASK>
__device__ __forceinline__ uint32_t dpp_k(uint32_t src) {
  return (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)src, CTRL, RMASK, 0xF, false);
}

template <int NV, int CTRL, int RMASK>
__device__ __forceinline__ void seg_step(float (&v)[NV], uint32_t key) {
  const uint32_t ks = dpp_k<CTRL, RMASK>(key);
  float t[NV];
#pragma unroll
  for (int q = 0; q < NV; ++q) t[q] = dpp_f<CTRL, RMASK>(v[q]);
  if (ks == key) {
#pragma unroll
    for (int q = 0; q < NV; ++q) v[q] += t[q];
  }
}

// Only the steps the chunk needs run (wave-uniform): with eq = lanes whose key equals the
// previous lane's, the longest run of set bits bounds the within-row shifts, and the
// row-crossing steps run only when a segment crosses lane 16/48 or 32.
template <int NV>
__device__ __forceinline__ void seg_scan(float (&v)[NV], uint32_t key) {
  // wave_shr:1
  const uint32_t kp = (uint32_t)__builtin_amdgcn_mov_dpp((int)key, 0x138, 0xF, 0xF, true);
  const int lane = threadIdx.x & 63;
  const uint64_t eq = __ballot(lane > 0 && kp == key);
  if (eq == 0) return;
  int run = 0;  // longest run of ones in eq
  for (uint64_t m = eq; m; m &= (m >> 1)) ++run;
  seg_step<NV, 0x111, 0xF>(v, key);                       // row_shr:1
  if (run >= 2) seg_step<NV, 0x112, 0xF>(v, key);         // row_shr:2
  if (run >= 4) seg_step<NV, 0x114, 0xF>(v, key);         // row_shr:4
  if (run >= 8) seg_step<NV, 0x118, 0xF>(v, key);         // row_shr:8
  if (eq & ((1ull << 16) | (1ull << 48))) seg_step<NV, 0x142, 0xA>(v, key);  // row_bcast:15
  if (eq & (1ull << 32)) seg_step<NV, 0x143, 0xC>(v, key);  // row_bcast:31
}

// The streams of one 64-particle chunk as they come from memory (one lane's particle).
template <int C>
struct RawChunk {
  uint32_t key;
  Vec3 f;
  Vec3 u;  // C = 3
  bool ok;
};

// Particles c0 .. c0 + 63 of the sorted stream, those in [beg, end) only.
template <int C>
__device__ __forceinline__ RawChunk<C> load_raw(const PaintArgs& a, uint32_t c0, uint32_t beg,
                                                uint32_t end) {
  const uint32_t j = c0 + (threadIdx.x & 63);
  RawChunk<C> r;
  r.ok = j >= beg && j < end;
  r.key = 0u;
  r.f = Vec3{0.f, 0.f, 0.f};
  r.u = Vec3{0.f, 0.f, 0.f};
  if (r.ok) {
    r.key = a.keys[j];
    r.f = a.frac[j];
    if constexpr (C == 3) r.u = a.val[j];
  }
  return r;
}

// One 64-particle chunk of a source run: per lane the four (oy, oz) weights of each channel.
template <int C>
struct Chunk {
  uint32_t key;
  int sy, iz;
  bool ok;
  float v[4 * C];
};

template <int C>
__device__ __forceinline__ void weigh_chunk(const PaintArgs& a, const RawChunk<C>& r, int ox,
                                            Chunk<C>& ch) {
  const int lane = threadIdx.x & 63;
  const int nm = a.nm;
  ch.ok = r.ok;
  ch.key = 0xffffffffu - lane;  // never equal across lanes when invalid
  ch.sy = 0;
  ch.iz = 0;
#pragma unroll
  for (int q = 0; q < 4 * C; ++q) ch.v[q] = 0.f;
  if (ch.ok) {
    const uint32_t key = r.key;
    const Vec3 f = r.f;
    ch.key = key;
    ch.iz = (int)(key & (uint32_t)(nm - 1));
    ch.sy = (int)((key >> a.log_nm) & (uint32_t)(nm - 1));
    const float wx = ox ? f.x : 1.f - f.x;
    float val[C];
    if constexpr (C == 1) {
      val[0] = a.mass * wx;
    } else {
      val[0] = r.u.x * wx;
      val[1] = r.u.y * wx;
      val[2] = r.u.z * wx;
    }
    const float wy0 = 1.f - f.y, wy1 = f.y, wz0 = 1.f - f.z, wz1 = f.z;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      ch.v[4 * c + 0] = val[c] * wy0 * wz0;
      ch.v[4 * c + 1] = val[c] * wy0 * wz1;
      ch.v[4 * c + 2] = val[c] * wy1 * wz0;
      ch.v[4 * c + 3] = val[c] * wy1 * wz1;
    }
  }
}

// Last lane of each run adds the run's sums to its two target rows. The accumulator is
// private to the wavefront and, within one phase below, the tails of a chunk touch
// distinct words, so a plain read-add-write is race-free inside a phase. Different phases
// (and chunks) may touch the same word from different lanes: a compiler barrier keeps the
// phases in program order, and LDS instructions of one wavefront execute in issue order,
// so every word receives its additions in one fixed order. (LDS float atomics without a
// return, in the same phases, would spare the read's wait; they measured 2-4.5 times slower
// for the whole paint.)
#define PMR_PHASE_FENCE() asm volatile("" ::: "memory")

// Float slot of cell iz in an LDS row: plain (iz), or, for rows that the z-pass FFT then
// transforms in place, the padded complex layout (one spare complex slot every 32 complex
// values: real point iz is half of complex point iz / 2).
template <bool PAD>
__device__ __forceinline__ int row_slot(int iz) {
  if constexpr (PAD) {
    const int k = iz >> 1;
    return 2 * (k + (k >> 5)) + (iz & 1);
  }
  return iz;
}

// acc rows: [TY][C] rows of rp floats each.
template <int C, int TY, bool PAD = false>
__device__ __forceinline__ void deposit(const Chunk<C>& ch, float* acc, int nm, int iy0, int rp) {
  const int lane = threadIdx.x & 63;
  // wave_shl:1
  const uint32_t kn = (uint32_t)__builtin_amdgcn_mov_dpp((int)ch.key, 0x130, 0xF, 0xF, true);
  const int ok_next = __builtin_amdgcn_mov_dpp((int)ch.ok, 0x130, 0xF, 0xF, true);
  const bool tail = ch.ok && (lane == 63 || !ok_next || kn != ch.key);
  const int iz1 = (ch.iz + 1) & (nm - 1);
#pragma unroll
  for (int ph = 0; ph < 4; ++ph) {
    const int oy = ph >> 1, oz = ph & 1;
    const int jt = ((ch.sy + oy) & (nm - 1)) - iy0;
    PMR_PHASE_FENCE();
    if (tail && jt >= 0 && jt < TY) {
      float* row = acc + (size_t)jt * C * rp + row_slot<PAD>(oz ? iz1 : ch.iz);
#pragma unroll
      for (int c = 0; c < C; ++c) row[c * rp] = row[c * rp] + ch.v[4 * c + 2 * oy + oz];
    }
    PMR_PHASE_FENCE();
  }
}

// One target row per wavefront (TY = 1): a particle of source row sy reaches that row
// through one corner row only (oy = 1 from row iy0 - 1, oy = 0 from row iy0; its other
// corner row belongs to another wavefront), so a chunk carries the 2 C values of that oy:
// half the weights and half the scan of the general chunk. The same lanes deposit the same
// values in the same phases as the general path, so the rows are bitwise the same.
template <int C>
struct Chunk1 {
  uint32_t key;
  int iz, oy;
  bool ok;
  float v[2 * C];
};

template <int C>
__device__ __forceinline__ void weigh_chunk1(const PaintArgs& a, const RawChunk<C>& r, int ox,
                                             int iy0, Chunk1<C>& ch) {
  const int lane = threadIdx.x & 63;
  const int nm = a.nm;
  ch.ok = r.ok;
  ch.key = 0xffffffffu - lane;  // never equal across lanes when invalid
  ch.iz = 0;
  ch.oy = 0;
#pragma unroll
  for (int q = 0; q < 2 * C; ++q) ch.v[q] = 0.f;
  if (ch.ok) {
    const uint32_t key = r.key;
    const Vec3 f = r.f;
    ch.key = key;
    ch.iz = (int)(key & (uint32_t)(nm - 1));
    const int sy = (int)((key >> a.log_nm) & (uint32_t)(nm - 1));
    ch.oy = sy == iy0 ? 0 : 1;
    const float wx = ox ? f.x : 1.f - f.x;
    float val[C];
    if constexpr (C == 1) {
      val[0] = a.mass * wx;
    } else {
      val[0] = r.u.x * wx;
      val[1] = r.u.y * wx;
      val[2] = r.u.z * wx;
    }
    const float wy = ch.oy ? f.y : 1.f - f.y, wz0 = 1.f - f.z, wz1 = f.z;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      ch.v[2 * c + 0] = val[c] * wy * wz0;
      ch.v[2 * c + 1] = val[c] * wy * wz1;
    }
  }
}

template <int C, bool PAD = false>
__device__ __forceinline__ void deposit1(const Chunk1<C>& ch, float* acc, int nm, int rp) {
  const int lane = threadIdx.x & 63;
  // wave_shl:1
  const uint32_t kn = (uint32_t)__builtin_amdgcn_mov_dpp((int)ch.key, 0x130, 0xF, 0xF, true);
  const int ok_next = __builtin_amdgcn_mov_dpp((int)ch.ok, 0x130, 0xF, 0xF, true);
  const bool tail = ch.ok && (lane == 63 || !ok_next || kn != ch.key);
  const int iz1 = (ch.iz + 1) & (nm - 1);
#pragma unroll
  for (int ph = 0; ph < 4; ++ph) {
    const int oy = ph >> 1, oz = ph & 1;
    PMR_PHASE_FENCE();
    if (tail && ch.oy == oy) {
      float* row = acc + row_slot<PAD>(oz ? iz1 : ch.iz);
#pragma unroll
      for (int c = 0; c < C; ++c) row[c * rp] = row[c * rp] + ch.v[2 * c + oz];
    }
    PMR_PHASE_FENCE();
  }
}

// Deposits of all particles that reach the TY target rows [iy0, iy0 + TY) of plane ix of one
// item, into the wavefront's rows acc (zeroed by the caller): the two source planes ix - 1
// and ix, each as one or two contiguous runs of source rows. Chunks are deposited in stream
// order; the streams of the next one are loaded before the current one is scanned, also from
// one run to the next, so that a wavefront's walk does not wait for memory at every chunk.
//
// The chunks are cut as if the wavefront owned the whole group of a.group (>= TY, a power of
// two) target rows that its rows lie in: the scan of a run of equal cells depends on where in
// its chunk the run lies, so a group's rows come out bitwise the same whether one wavefront
// owns them all or several share them. Sharing shortens each wavefront's serial walk of
// dependent chunks at the price of reading the chunks at the seams more than once.
template <int C, int TY, bool PAD = false>
__device__ __forceinline__ void paint_rows(const PaintArgs& a, int item, int ix, int iy0,
                                           float* acc, int rp) {
  const int nm = a.nm;
  const int rows_item = item * nm * nm;
  // main runs of source rows [iy0 - 1, iy0 + TY - 1] of both planes (from row 0 when iy0 - 1
  // wraps; row nm - 1 is then a second run), and the first source row of the group's run
  const int lo0 = iy0 == 0 ? 0 : iy0 - 1, hi0 = iy0 + TY - 1;
  const int g0 = iy0 & ~(a.group - 1);
  const int glo = g0 == 0 ? 0 : g0 - 1;
  const uint32_t* rs0 = a.row_start + rows_item + ix * nm;
  const uint32_t* rs1 = a.row_start + rows_item + ((ix - 1 + nm) & (nm - 1)) * nm;
  // one run of the walk: its first chunk, its particles [beg, end); scalar registers, so that
  // the walk itself costs no vector instructions
  struct Run {
    uint32_t cut, beg, end;
  };
  auto uni = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };
  uint32_t v[10] = {rs0[glo], rs0[lo0], rs0[hi0 + 1], rs1[glo], rs1[lo0], rs1[hi0 + 1], 0, 0, 0, 0};
  if (iy0 == 0) {
    v[6] = rs0[nm - 1];
    v[7] = rs0[nm];
    v[8] = rs1[nm - 1];
    v[9] = rs1[nm];
  }
#pragma unroll
  for (int i = 0; i < 10; ++i) v[i] = uni(v[i]);
  auto main_run = [](uint32_t g, uint32_t b, uint32_t e) {
    return Run{b == e ? e : g + ((b - g) & ~63u), b, e};
  };
  Run now = main_run(v[0], v[1], v[2]), n1 = Run{v[6], v[6], v[7]};
  Run n2 = main_run(v[3], v[4], v[5]), n3 = Run{v[8], v[8], v[9]};
  int run = 0;  // 0, 1: source plane ix; 2, 3: ix - 1
  uint32_t c0 = now.cut;
  auto settle = [&]() {  // on to the next run while this one is done; false after the last
    while (c0 >= now.end) {
      if (run == 3) return false;
      ++run;
      now = n1;
      n1 = n2;
      n2 = n3;
      c0 = now.cut;
    }
    return true;
  };
  bool more = settle();
  RawChunk<C> next;
  if (more) next = load_raw<C>(a, c0, now.beg, now.end);
#pragma unroll 1
  while (more) {
    const RawChunk<C> cur = next;
    const int ox = run >> 1;
    c0 += 64;
    more = settle();
    if (more) next = load_raw<C>(a, c0, now.beg, now.end);
    if constexpr (TY == 1) {
      Chunk1<C> ch;
      weigh_chunk1<C>(a, cur, ox, iy0, ch);
      seg_scan<2 * C>(ch.v, ch.key);
      deposit1<C, PAD>(ch, acc, nm, rp);
    } else {
      Chunk<C> ch;
      weigh_chunk<C>(a, cur, ox, ch);
      seg_scan<4 * C>(ch.v, ch.key);
      deposit<C, TY, PAD>(ch, acc, nm, iy0, rp);
    }
  }
}
