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

// The same step for finite values in one instruction per value: v = t * m + v with m = 1 where
// the source lane is in my segment and 0 elsewhere, the lane move being the operand's. With
// m = 1 the product is exact, so the sum rounds as the plain addition does; with m = 0 a finite
// v is unchanged (a -0 may become +0, which no sum that starts at +0 can tell apart). The
// paints are bound by their vector instructions, half of which these steps were: with them, the
// branch-free loads and the lane masks in scalar registers a chunk of 3 channels went from
// about 250 to 165, and a launch (us, before -> now) from 54.9 to 43.4 (3 channels) and 35.8 to
// 28.1 (1) at 128^3, 156 to 145 and 82 to 69 at 64^3 x 32, 836 to 803 and 308 to 291 for 256^3 on
// 512^3; unfused, 57 to 33 at 128^3, 113 to 77 at 64^3 x 32 and 318 to 167 at 256^3.
// The compiler does not see into the block, so the wait states between a vector write and a
// lane move's read of it stand in it. Rows out of RMASK keep v.
template <int CTRL>
__device__ __forceinline__ void fma_move4(float& a, float& b, float& c, float& d, float m) {
#define PMR_FMA_MOVE4(MOVE)                               \
  asm volatile("s_nop 1\n\t"                              \
               "v_fmac_f32_dpp %0, %0, %4 " MOVE "\n\t"   \
               "v_fmac_f32_dpp %1, %1, %4 " MOVE "\n\t"   \
               "v_fmac_f32_dpp %2, %2, %4 " MOVE "\n\t"   \
               "v_fmac_f32_dpp %3, %3, %4 " MOVE          \
               : "+v"(a), "+v"(b), "+v"(c), "+v"(d)       \
               : "v"(m))
  if constexpr (CTRL == 0x111) PMR_FMA_MOVE4("row_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:0");
  if constexpr (CTRL == 0x112) PMR_FMA_MOVE4("row_shr:2 row_mask:0xf bank_mask:0xf bound_ctrl:0");
  if constexpr (CTRL == 0x114) PMR_FMA_MOVE4("row_shr:4 row_mask:0xf bank_mask:0xf bound_ctrl:0");
  if constexpr (CTRL == 0x118) PMR_FMA_MOVE4("row_shr:8 row_mask:0xf bank_mask:0xf bound_ctrl:0");
  if constexpr (CTRL == 0x142) PMR_FMA_MOVE4("row_bcast:15 row_mask:0xa bank_mask:0xf");
  if constexpr (CTRL == 0x143) PMR_FMA_MOVE4("row_bcast:31 row_mask:0xc bank_mask:0xf");
#undef PMR_FMA_MOVE4
}

// (A lane without a source reads key 0 and value 0, which it may add; a row out of the move's
// mask may compare anything.)
template <int NV, int CTRL>
__device__ __forceinline__ void seg_step_fma(float (&v)[NV], uint32_t key) {
  const uint32_t ks = (uint32_t)__builtin_amdgcn_mov_dpp((int)key, CTRL, 0xF, 0xF, true);
  const float m = ks == key ? 1.f : 0.f;
  static_assert(NV % 2 == 0, "");
#pragma unroll
  for (int q = 0; q + 4 <= NV; q += 4) fma_move4<CTRL>(v[q], v[q + 1], v[q + 2], v[q + 3], m);
  if constexpr (NV % 4 == 2) {
    float p0 = 0.f, p1 = 0.f;
    fma_move4<CTRL>(v[NV - 2], v[NV - 1], p0, p1, m);
  }
}

// Only the steps the chunk needs run (wave-uniform): bit i of eq says that lane i continues the
// run of lane i - 1. A shift by k inside the rows adds something only where k such bits follow one
// another within a row; the row-crossing steps only where a segment crosses lane 16/48 or 32.
template <int NV, bool FMA>
__device__ __forceinline__ void seg_scan_steps(float (&v)[NV], uint32_t key, uint64_t eq) {
#define PMR_SEG_STEP(CTRL, RMASK)              \
  do {                                         \
    if constexpr (FMA)                         \
      seg_step_fma<NV, CTRL>(v, key);          \
    else                                       \
      seg_step<NV, CTRL, RMASK>(v, key);       \
  } while (0)
  const uint64_t r1 = eq & 0xFFFEFFFEFFFEFFFEull;
  if (r1) {
    PMR_SEG_STEP(0x111, 0xF);  // row_shr:1
    const uint64_t r2 = r1 & (r1 >> 1);
    if (r2) {
      PMR_SEG_STEP(0x112, 0xF);  // row_shr:2
      const uint64_t r4 = r2 & (r2 >> 2);
      if (r4) {
        PMR_SEG_STEP(0x114, 0xF);                      // row_shr:4
        if (r4 & (r4 >> 4)) PMR_SEG_STEP(0x118, 0xF);  // row_shr:8
      }
    }
  }
  if (eq & ((1ull << 16) | (1ull << 48))) PMR_SEG_STEP(0x142, 0xA);  // row_bcast:15
  if (eq & (1ull << 32)) PMR_SEG_STEP(0x143, 0xC);                   // row_bcast:31
#undef PMR_SEG_STEP
}

// Scans v over the runs of equal keys and returns the lanes, of those in `ok`, that end a run
// (two valid lanes only ever share a key with valid lanes between them; what a lane without a
// particle, whose key is its neighbour's, adds to a valid one is 0, and those above the run are no
// valid lane's source).
// `tame`: this lane's values and all sums of up to 64 like them are finite.
template <int NV>
__device__ __forceinline__ uint64_t seg_scan(float (&v)[NV], uint32_t key, uint64_t ok,
                                             bool tame) {
  // wave_shr:1
  const uint32_t kp = (uint32_t)__builtin_amdgcn_mov_dpp((int)key, 0x138, 0xF, 0xF, true);
  const uint64_t eq = run_joins(__ballot(kp == key), ok);
  if (eq != 0) {
    uint64_t wild = __ballot(!tame);
    if (wild == 0) seg_scan_steps<NV, true>(v, key, eq);
    asm volatile("" : "+s"(wild));  // two branches, not two arms: both scan v in place
    if (wild != 0) {
      if (!__builtin_amdgcn_inverse_ballot_w64(ok)) {
#pragma unroll
        for (int q = 0; q < NV; ++q) v[q] = 0.f;  // (0 times a neighbour's NaN)
      }
      seg_scan_steps<NV, false>(v, key, eq);
    }
  }
  return run_ends(eq, ok);
}

// The streams of one 64-particle chunk as they come from memory (one lane's particle).
template <int C>
struct RawChunk {
  uint32_t key;
  Vec3 f;
  Vec3 u;  // C = 3
  uint64_t ok;  // lanes with a particle of the run (uniform)
};

// Particles c0 .. c0 + 63 of the sorted stream, those in [beg, end) only (at least one). The
// other lanes read the run's first or last particle of the chunk, so that the loads need no
// branch and, from a uniform base, no 64-bit address per lane; the weights drop them.
template <int C>
__device__ __forceinline__ RawChunk<C> load_raw(const PaintArgs& a, uint32_t c0, uint32_t beg,
                                                uint32_t end) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t lo = beg > c0 ? beg - c0 : 0u;
  const uint32_t hi = (end - c0 < 64u ? end - c0 : 64u) - 1u;
  const uint32_t l = lane < lo ? lo : lane > hi ? hi : lane;
  RawChunk<C> r;
  r.ok = (~0ull << lo) & (~0ull >> (63u - hi));
  r.key = (a.keys + c0)[l];
  r.f = (a.frac + c0)[l];
  r.u = Vec3{0.f, 0.f, 0.f};
  if constexpr (C == 3) r.u = (a.val + c0)[l];
  return r;
}

// The C values of a lane's particle times its x weight, 0 on lanes without one, and whether
// sums of 64 such values times further weights stay finite.
template <int C>
__device__ __forceinline__ bool chunk_values(const PaintArgs& a, const RawChunk<C>& r, int ox,
                                             bool ok, float (&val)[C]) {
  const float wx = ox ? r.f.x : 1.f - r.f.x;
  float mag = r.f.y + r.f.z;  // in [0, 2], or NaN
  if constexpr (C == 1) {
    val[0] = (ok ? a.mass : 0.f) * wx;
  } else {
    val[0] = (ok ? r.u.x : 0.f) * wx;
    val[1] = (ok ? r.u.y : 0.f) * wx;
    val[2] = (ok ? r.u.z : 0.f) * wx;
  }
#pragma unroll
  for (int c = 0; c < C; ++c) mag += fabsf(val[c]);
  return mag < 0x1p120f;
}

// One 64-particle chunk of a source run: per lane the four (oy, oz) weights of each channel.
template <int C>
struct Chunk {
  uint32_t key;
  int sy, iz;
  uint64_t ok;
  bool tame;
  float v[4 * C];
};

template <int C>
__device__ __forceinline__ void weigh_chunk(const PaintArgs& a, const RawChunk<C>& r, int ox,
                                            Chunk<C>& ch) {
  const int nm = a.nm;
  const bool ok = __builtin_amdgcn_inverse_ballot_w64(r.ok);
  const Vec3 f = r.f;
  ch.ok = r.ok;
  ch.key = r.key;
  ch.iz = (int)(r.key & (uint32_t)(nm - 1));
  ch.sy = (int)((r.key >> a.log_nm) & (uint32_t)(nm - 1));
  float val[C];
  ch.tame = chunk_values<C>(a, r, ox, ok, val);
  const float wy0 = 1.f - f.y, wy1 = f.y, wz0 = 1.f - f.z, wz1 = f.z;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    ch.v[4 * c + 0] = val[c] * wy0 * wz0;
    ch.v[4 * c + 1] = val[c] * wy0 * wz1;
    ch.v[4 * c + 2] = val[c] * wy1 * wz0;
    ch.v[4 * c + 3] = val[c] * wy1 * wz1;
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
    return iz + 2 * (iz >> 6);
  }
  return iz;
}

// acc rows: [TY][C] rows of rp floats each; tails: the lanes that end a run.
template <int C, int TY, bool PAD = false>
__device__ __forceinline__ void deposit(const Chunk<C>& ch, uint64_t tails, float* acc, int nm,
                                        int iy0, int rp) {
  const bool tail = __builtin_amdgcn_inverse_ballot_w64(tails);
  const int slot[2] = {row_slot<PAD>(ch.iz), row_slot<PAD>((ch.iz + 1) & (nm - 1))};
#pragma unroll
  for (int ph = 0; ph < 4; ++ph) {
    const int oy = ph >> 1, oz = ph & 1;
    const uint32_t jt = (uint32_t)(((ch.sy + oy) & (nm - 1)) - iy0);
    PMR_PHASE_FENCE();
    if (tail && jt < (uint32_t)TY) {
      float* row = acc + __umul24(jt, C * rp) + slot[oz];
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
  uint64_t ok;
  bool tame;
  float v[2 * C];
};

template <int C>
__device__ __forceinline__ void weigh_chunk1(const PaintArgs& a, const RawChunk<C>& r, int ox,
                                             int iy0, Chunk1<C>& ch) {
  const int nm = a.nm;
  const bool ok = __builtin_amdgcn_inverse_ballot_w64(r.ok);
  const Vec3 f = r.f;
  ch.ok = r.ok;
  ch.key = r.key;
  ch.iz = (int)(r.key & (uint32_t)(nm - 1));
  ch.oy = (int)((r.key >> a.log_nm) & (uint32_t)(nm - 1)) == iy0 ? 0 : 1;
  float val[C];
  ch.tame = chunk_values<C>(a, r, ox, ok, val);
  const float wy = ch.oy ? f.y : 1.f - f.y, wz0 = 1.f - f.z, wz1 = f.z;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    ch.v[2 * c + 0] = val[c] * wy * wz0;
    ch.v[2 * c + 1] = val[c] * wy * wz1;
  }
}

template <int C, bool PAD = false>
__device__ __forceinline__ void deposit1(const Chunk1<C>& ch, uint64_t tails, float* acc, int nm,
                                         int rp) {
  const bool tail = __builtin_amdgcn_inverse_ballot_w64(tails);
  const int slot[2] = {row_slot<PAD>(ch.iz), row_slot<PAD>((ch.iz + 1) & (nm - 1))};
#pragma unroll
  for (int ph = 0; ph < 4; ++ph) {
    const int oy = ph >> 1, oz = ph & 1;
    PMR_PHASE_FENCE();
    if (tail && ch.oy == oy) {
      float* row = acc + slot[oz];
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
      const uint64_t tails = seg_scan<2 * C>(ch.v, ch.key, ch.ok, ch.tame);
      deposit1<C, PAD>(ch, tails, acc, nm, rp);
    } else {
      Chunk<C> ch;
      weigh_chunk<C>(a, cur, ox, ch);
      const uint64_t tails = seg_scan<4 * C>(ch.v, ch.key, ch.ok, ch.tame);
      deposit<C, TY, PAD>(ch, tails, acc, nm, iy0, rp);
    }
  }
}
