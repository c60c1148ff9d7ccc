// Apply pass of section 3.1 as device functions over rows of one camera:
// every sample is blended between the identity and its side's affine map with
// the Q8 weight of its column, y = ((256 - w) x + w f(x) + 128) >> 8, in exact
// integers; optionally fused with the whole-frame histogram and sums of the
// input samples.
//
// A workgroup of kApplyThreads threads takes a run of rows.  Its threads lie
// over the image as ap_lanes rows of ap_cols groups of 4 consecutive pixels
// (12 bytes for RGB8, 4 for gray8, 8 for gray16); a thread keeps its columns
// and walks down the run ap_lanes rows at a time, rows_in_flight of them, so
// its pixels' weights and its side's map constants stay in registers.  Images
// whose groups do not fit the workgroup in one row, or fill it badly, are
// taken in column chunks (see lay_rows).  The maps
// of the run's blocks (or, blended between blocks, of its rows) are staged in
// LDS, kMapBytes at a time.  The histogram is kept in LDS in kRep replicas
// interleaved bin by bin, lane l updating replica l % kRep, so that lanes of
// one wave that see the same value mostly hit different LDS words; after the
// run the replicas are summed and added to the camera's whole-frame
// statistics with global atomics (the whole-frame buffers must be zero before
// the first run).
//
// The runs of a camera interleave (run i of m takes every m-th step of ap_lanes
// rows) where they hold enough rows for it, and are contiguous elsewhere (see
// runs_interleave).  The form that stages whole 256-entry tables, two blocks of
// RGB at a time, is always contiguous: rt_apply without statistics took, us
// interleaved and contiguous, 14x1920x1080 of 16 blocks 42.5 and 36.8, of 64
// blocks 75.6 and 37.2, 3x200x150 8.2 and 4.2.
//
// What bounds it: memory requests in flight and, next to them, the vector ALU
// and the LDS atomics, each busy about half of the time.  Long runs pay the
// set-up and the flush of the histogram once per half compute unit, and rows
// side by side keep narrow images' workgroups full.  Measured on MI355X (us,
// statistics fused; one 256-thread workgroup per 22-row tile, runs of
// neighbouring rows, interleaved runs): 14x1920x1080 RGB8, 174 MB, 50.6, 44.7,
// 43.0, and 42.0 with the present layout and registers.  1x640x480 18.5 by tiles
// and 9.3, 5x1031x517 RGB8 58.2 and 14.7, which was the ragged row ends, read
// byte by byte and row by row.
//
// Registers: at most 96 (RC_APPLY_WAVES 5) and none spilled, so that beside the
// four waves per SIMD of two workgroups a seam-estimate wave finds room; at 108
// the pipeline of the 14x1920x1080 rig took 258.8 us per six frame-sets, at 96
// 250.5, and without the six to eight spills of that form 5 us less (246.6 and
// 241.3 side by side).  The look-ahead launch holds to it too (97 with blended
// maps); 3x3 maps with statistics take 98.
#pragma once

#include <type_traits>

#include "dev_estimate.h"
#include "dev_stats.h"

namespace rc {

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x3 __attribute__((ext_vector_type(3)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

#ifndef RC_LOAD_POLICY
#define RC_LOAD_POLICY 2      // non-temporal: every frame byte is touched exactly once
#endif
#ifndef RC_STORE_POLICY
#define RC_STORE_POLICY 2
#endif
constexpr int kRep = 8;                        // histogram replicas
constexpr int kLoadPolicy = RC_LOAD_POLICY;    // cache-policy bits of frame loads
constexpr int kStorePolicy = RC_STORE_POLICY;  // cache-policy bits of frame stores

constexpr int kMapBytes = 3072;                // staged maps
constexpr int kMapEntries = kSplitBlocks;      // most blocks (or rows) staged at a time

struct ApplyLds {
  alignas(16) uint8_t map[kMapBytes];          // [block or row][side][channel] maps, see stage_maps
  alignas(16) uint32_t hist[kCS * kNB * kRep]; // [channel][bin][replica]
  int32_t end[kMapEntries];                    // first row after each staged block
  alignas(16) int32_t good[kApplyThreads / kWave];   // per wave, see stage_maps
  unsigned long long sums[9];                  // [channel] (n, S1, S2) of the run
};

template <int NW, int POL = kLoadPolicy>
__device__ inline void load_group(__amdgpu_buffer_rsrc_t r, int off, uint32_t (&d)[NW]) {
  if constexpr (NW == 3) {
    u32x3 v = __builtin_amdgcn_raw_buffer_load_b96(r, off, 0, POL);
    d[0] = v.x; d[1] = v.y; d[2] = v.z;
  } else if constexpr (NW == 2) {
    u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, POL);
    d[0] = v.x; d[1] = v.y;
  } else {
    d[0] = __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, POL);
  }
}

template <int NW, int POL = kStorePolicy>
__device__ inline void store_group(__amdgpu_buffer_rsrc_t r, int off, const uint32_t (&d)[NW]) {
  if constexpr (NW == 3) {
    u32x3 v = {d[0], d[1], d[2]};
    __builtin_amdgcn_raw_buffer_store_b96(v, r, off, 0, POL);
  } else if constexpr (NW == 2) {
    u32x2 v = {d[0], d[1]};
    __builtin_amdgcn_raw_buffer_store_b64(v, r, off, 0, POL);
  } else {
    __builtin_amdgcn_raw_buffer_store_b32(d[0], r, off, 0, POL);
  }
}

// The first nb (1 .. 4 NW) bytes of a group at the ragged end of a row, whole
// dwords first, then the rest: no byte beyond the row is touched.
template <int NW>
__device__ inline void load_part(__amdgpu_buffer_rsrc_t r, int off, int nb, uint32_t (&d)[NW]) {
#pragma unroll
  for (int q = 0; q < NW; ++q) {
    const int rem = nb - 4 * q;
    d[q] = 0;
    if (rem >= 4) d[q] = __builtin_amdgcn_raw_buffer_load_b32(r, off + 4 * q, 0, 0);
    else if (rem >= 2) {
      d[q] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, off + 4 * q, 0, 0);
      if (rem == 3) d[q] |= (uint32_t)(uint8_t)__builtin_amdgcn_raw_buffer_load_b8(r, off + 4 * q + 2, 0, 0) << 16;
    } else if (rem == 1) d[q] = (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(r, off + 4 * q, 0, 0);
  }
}

template <int NW>
__device__ inline void store_part(__amdgpu_buffer_rsrc_t r, int off, int nb, const uint32_t (&d)[NW]) {
#pragma unroll
  for (int q = 0; q < NW; ++q) {
    const int rem = nb - 4 * q;
    if (rem >= 4) __builtin_amdgcn_raw_buffer_store_b32(d[q], r, off + 4 * q, 0, 0);
    else if (rem >= 2) {
      __builtin_amdgcn_raw_buffer_store_b16((uint16_t)d[q], r, off + 4 * q, 0, 0);
      if (rem == 3) __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(d[q] >> 16), r, off + 4 * q + 2, 0, 0);
    } else if (rem == 1) __builtin_amdgcn_raw_buffer_store_b8((uint8_t)d[q], r, off + 4 * q, 0, 0);
  }
}

// How a run's maps are staged and evaluated, f(x) = clamp((A x + Bq + 2^15) >> 16):
//   kMapDirect  32-bit integers: (A, Bq + 2^15) as int32, for 8-bit samples whose
//               maps pass small_map;
//   kMapWide    64-bit integers: (A, Bq) as int64;
//   kMapTable   the caller's 256-entry tables (8-bit samples);
//   kMapCross / kMapCrossWide  3x3 maps across the channels, f_r(x) =
//               clamp((A_r . x + B_r + 2^15) >> 16, 0, 255), in 32-bit integers
//               (B_r + 2^15 staged) or 64-bit ones.
constexpr int kX3 = 12;   // parameters of one 3x3 map

template <int KIND, int C>
struct MapEntry {   // bytes of one block's (or row's) staged maps, both sides
  static constexpr int kBytes = KIND == kMapDirect ? 2 * C * 8 : KIND == kMapWide ? 2 * C * 16
                                : KIND == kMapTable ? 2 * C * kNB : KIND == kMapCross ? 2 * kX3 * 4 : 2 * kX3 * 8;
  static constexpr int kCap = kMapBytes / kBytes < kMapEntries ? kMapBytes / kBytes : kMapEntries;
};

// An 8-bit map may be evaluated directly, bit for bit equal to its table, when
// A fits a 24-bit multiply and A x + Bq + 2^15 stays inside int32 for x in [0,
// 255].
__device__ inline bool small_map(int64_t A, int64_t Bq) {
  const int64_t c = Bq + 32768, e = 255 * A + c;
  return A < (1 << 23) && A >= -(1 << 23) && c <= INT32_MAX && c >= INT32_MIN && e <= INT32_MAX && e >= INT32_MIN;
}

// Row-wise blend of adjacent blocks' maps (section 5's convex combinations of
// the maps of adjacent blocks; every block holds at least one row): with
// doubled block centres C_j = r0_j + r1_j - 1, row r of block j blends j with
// its neighbour on r's side of the centre (alone before the first and from
// the last centre on), weight v of the second block = round_half_up(256
// (2r - C_a) / (C_b - C_a)); each Q16 parameter of the row is
// floor(((256 - v) P_a + v P_b + 128) / 256).
// First row of block j, and the block that holds row r (products stay below
// 2^26: at most 32768 rows and 1024 blocks).
__device__ inline int block_row(int j, int H, int nb) { return (int)((uint32_t)j * (uint32_t)H / (uint32_t)nb); }
__device__ inline int row_block(int r, int H, int nb) {
  return (int)(((uint32_t)(r + 1) * (uint32_t)nb - 1u) / (uint32_t)H);
}
__device__ inline int block_centre2(int j, int H, int nb) { return block_row(j, H, nb) + block_row(j + 1, H, nb) - 1; }

__device__ inline void vblend_row(int H, int nb, int r, int& a, int& b, int& v) {
  const int j = row_block(r, H, nb);
  const int lo = 2 * r < block_centre2(j, H, nb) ? j - 1 : j;
  if (lo < 0 || lo + 1 >= nb) {
    a = b = j;
    v = 0;
    return;
  }
  const int ca = block_centre2(lo, H, nb), cb = block_centre2(lo + 1, H, nb);
  a = lo;
  b = lo + 1;
  v = ((2 * r - ca) * 512 + (cb - ca)) / (2 * (cb - ca));
}

__device__ inline int64_t blend_q16(int64_t pa, int64_t pb, int v) {
  return ((256 - v) * pa + v * pb + 128) >> 8;
}

// Row r of a 3x3 map q: coefficients that fit 24-bit multiplies, and A_r . x +
// B_r + 2^15 inside int32 for every x in [0, 255]^3.
__device__ inline bool small_cross(const int64_t* q, int r) {
  int64_t lo = q[9 + r] + 32768, hi = lo;
  bool ok = lo <= INT32_MAX && lo >= INT32_MIN;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const int64_t a = q[r * 3 + c];
    const bool fits = a < (1 << 23) && a > -(1 << 23);
    ok = ok && fits;
    lo += fits && a < 0 ? 255 * a : 0;
    hi += fits && a > 0 ? 255 * a : 0;
  }
  return ok && lo >= INT32_MIN && hi <= INT32_MAX;
}

// Stages the maps of a piece of the run: entry e is block j0 + e, or with VB
// the run's row p0 + (e / lanes) stride + e % lanes (its two blocks' maps
// blended).  Ends with a barrier and returns the number of entries, from the
// first on, that the form evaluates exactly: fewer than n only where 32-bit
// arithmetic does not hold a map.  That is looked at on the values on their way
// to LDS; a pass over them of its own took 0.4 us more of every workgroup.
template <int C, int BPS, int KIND, bool VB>
__device__ inline int stage_maps(const Geo& g, const Bufs& b, const int64_t* q3, const DevCam& cam, int k, int p0,
                                 int stride, int j0, int n, ApplyLds& L, int tid) {
  const int nb = g.n_blocks, H = cam.height;
  constexpr int kPer = KIND == kMapTable ? 2 * C * kNB / 4 : KIND >= kMapCross ? 2 * kX3 : 2 * C;
  int good = n;
  if (!VB && tid < n) L.end[tid] = block_row(j0 + tid + 1, H, nb);
  for (int i = tid; i < n * kPer; i += kApplyThreads) {
    const int e = i / kPer, rem = i - e * kPer;
    if constexpr (KIND == kMapTable) {
      constexpr int kSide = C * kNB / 4;
      const int s = rem / kSide;
      const uint32_t* src =
          reinterpret_cast<const uint32_t*>(b.lut8 + unit_index(k, s, j0 + e, 0, nb) * kNB);
      reinterpret_cast<uint32_t*>(L.map)[i] = src[rem - s * kSide];
    } else if constexpr (KIND >= kMapCross) {
      const int s = rem / kX3, q = rem - s * kX3;
      const int64_t v = q3[(((int64_t)k * 2 + s) * nb + j0 + e) * kX3 + q];
      if (KIND == kMapCross) reinterpret_cast<int32_t*>(L.map)[i] = (int32_t)(q < 9 ? v : v + 32768);
      else reinterpret_cast<int64_t*>(L.map)[i] = v;
    } else {
      const int s = rem / C, c = rem - s * C;
      int64_t A, B;
      if (VB) {
        int ja, jb, v;
        vblend_row(H, nb, min(H - 1, p0 + (e / cam.ap_lanes) * stride + e % cam.ap_lanes), ja, jb, v);
        const int64_t ua = unit_index(k, s, ja, c, nb), ub = unit_index(k, s, jb, c, nb);
        A = blend_q16(b.q16[ua * 2], b.q16[ub * 2], v);
        B = blend_q16(b.q16[ua * 2 + 1], b.q16[ub * 2 + 1], v);
      } else {
        const int64_t u = unit_index(k, s, j0 + e, c, nb);
        A = b.q16[u * 2];
        B = b.q16[u * 2 + 1];
      }
      if (KIND == kMapDirect) {
        if (!small_map(A, B)) good = min(good, e);
        reinterpret_cast<int32_t*>(L.map)[2 * i] = (int32_t)A;
        reinterpret_cast<int32_t*>(L.map)[2 * i + 1] = (int32_t)(B + 32768);
      } else {
        reinterpret_cast<int64_t*>(L.map)[2 * i] = A;
        reinterpret_cast<int64_t*>(L.map)[2 * i + 1] = B;
      }
    }
  }
  if constexpr (KIND == kMapDirect || KIND == kMapCross) {
    if (KIND == kMapCross)
      for (int i = tid; i < n * 6; i += kApplyThreads) {
        const int e = i / 6, s = i / 3 & 1;
        if (!small_cross(q3 + (((int64_t)k * 2 + s) * nb + j0 + e) * kX3, i % 3)) good = min(good, e);
      }
    if (__builtin_amdgcn_ballot_w64(good < n) != 0) {
#pragma unroll
      for (int o = kWave / 2; o; o >>= 1) good = min(good, __shfl_xor(good, o, kWave));
    }
    if (tid % kWave == 0) L.good[tid / kWave] = good;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kApplyThreads / kWave; ++w) good = min(good, L.good[w]);
    return uniform((int32_t)good);
  }
  __syncthreads();
  return n;
}

// The maps of one side of one entry, in registers (the tables stay in LDS).
template <int C, int KIND>
struct SideMap {
  static constexpr int kN = KIND >= kMapCross ? kX3 : 2 * C;
  int32_t v[KIND == kMapDirect || KIND == kMapCross ? kN : 1];
  int64_t w[KIND == kMapWide || KIND == kMapCrossWide ? kN : 1];
  const uint8_t* t;

  __device__ inline void read(const ApplyLds& L, int entry, int side) {
    const int at = (entry * 2 + side) * (MapEntry<KIND, C>::kBytes / 2);
    if constexpr (KIND == kMapDirect || KIND == kMapCross) {
#pragma unroll
      for (int i = 0; i < kN; ++i) v[i] = reinterpret_cast<const int32_t*>(L.map + at)[i];
    } else if constexpr (KIND == kMapTable) {
      t = L.map + at;
    } else {
#pragma unroll
      for (int i = 0; i < kN; ++i) w[i] = reinterpret_cast<const int64_t*>(L.map + at)[i];
    }
  }

  // x | f_c(x) << 16 for channel c of the pixel's samples xs.
  __device__ inline uint32_t pair(const uint32_t (&xs)[C], int c, uint32_t maxv) const {
    const uint32_t x = xs[c];
    if constexpr (KIND == kMapDirect || KIND == kMapCross) {
      // Staged coefficients fit 24 bits (small_map), so these are 24-bit
      // multiplies.  clamp(v >> 16, 0, 255) << 16 == clamp(v, 0, 2^24 - 1) &
      // 0xffff0000 for the arithmetic shift, so f lands in the high half.
      // The whole sum is inside int32, its parts may not be.
      auto m24 = [](int32_t a, uint32_t s) { return (uint32_t)(((int32_t)((uint32_t)a << 8) >> 8) * (int32_t)s); };
      int32_t y;
      if constexpr (KIND == kMapDirect) {
        y = (int32_t)(m24(v[2 * c], x) + (uint32_t)v[2 * c + 1]);
      } else {
        y = (int32_t)(m24(v[c * 3], xs[0]) + m24(v[c * 3 + 1], xs[C > 1 ? 1 : 0]) +
                      m24(v[c * 3 + 2], xs[C > 2 ? 2 : 0]) + (uint32_t)v[9 + c]);
      }
      y = y < 0 ? 0 : (y > 0xffffff ? 0xffffff : y);
      return ((uint32_t)y & 0xffff0000u) | x;
    } else if constexpr (KIND == kMapTable) {
      return x | ((uint32_t)t[c * kNB + x] << 16);
    } else {
      int64_t y;
      if constexpr (KIND == kMapWide) {
        y = (w[2 * c] * (int64_t)x + w[2 * c + 1] + 32768) >> 16;
      } else {
        y = (w[c * 3] * (int64_t)xs[0] + w[c * 3 + 1] * (int64_t)xs[C > 1 ? 1 : 0] +
             w[c * 3 + 2] * (int64_t)xs[C > 2 ? 2 : 0] + w[9 + c] + 32768) >> 16;
      }
      y = y < 0 ? 0 : (y > (int64_t)maxv ? (int64_t)maxv : y);
      return x | ((uint32_t)y << 16);
    }
  }
};

// Four raw dot products (see one_group) to one dword of 8-bit samples: byte 1
// of each, in order, by two byte permutes (selector byte 0x0c gives zero).
__device__ inline uint32_t pack_raw4(uint32_t r0, uint32_t r1, uint32_t r2, uint32_t r3) {
  return __builtin_amdgcn_perm(r1, r0, 0x0c0c0501u) | __builtin_amdgcn_perm(r3, r2, 0x05010c0cu);
}

// 16-bit sample sums of a thread (S1, S2; 8-bit sums follow from the histogram).
struct Sums16 {
  unsigned long long s1, s2;
};

// One row of a 4-pixel group: histogram of its first npx pixels' samples
// (STATS) and their corrected values (WRITE) with the maps m; wp[p] is pixel
// p's weight pair (256 - w, w).
template <int C, int BPS, bool WRITE, bool STATS, class Map>
__device__ inline void one_group(const uint32_t (&d)[C * BPS], uint32_t (&o)[C * BPS], int npx, const Map& m,
                                 const uint32_t (&wp)[4], ApplyLds& L, int hrep, int shift, uint32_t maxv,
                                 Sums16& sums) {
  uint32_t r[4 * C];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    uint32_t xs[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int i = p * C + c;
      if (BPS == 1) xs[c] = (d[i >> 2] >> (8 * (i & 3))) & 0xffu;
      else xs[c] = (d[i >> 1] >> (16 * (i & 1))) & 0xffffu;
      if (STATS && p < npx) {
        uint32_t bin = xs[c];
        if (BPS == 2) {
          bin >>= shift;
          bin = bin > 255u ? 255u : bin;
          sums.s1 += xs[c];
          sums.s2 += (unsigned long long)xs[c] * xs[c];
        }
        __hip_atomic_fetch_add(&L.hist[(c * kNB + bin) * kRep + hrep], 1u, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
    if (WRITE) {
#pragma unroll
      for (int c = 0; c < C; ++c)
        // ((256 - w) x + w f + 128) >> 8 as one dot product of (x, f) with
        // (256 - w, w): the sum stays below 2^16 for 8-bit samples, byte 1 is y.
        r[p * C + c] = __builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, m.pair(xs, c, maxv)),
                                              __builtin_bit_cast(u16x2, wp[p]), 128u, false);
    }
  }
  if (WRITE) {
#pragma unroll
    for (int q = 0; q < C * BPS; ++q) {
      if (BPS == 1) o[q] = pack_raw4(r[4 * q], r[4 * q + 1], r[4 * q + 2], r[4 * q + 3]);
      else o[q] = ((r[2 * q] >> 8) & 0xffffu) | ((r[2 * q + 1] >> 8) << 16);
    }
  }
}

// The run's rows in [p0, p1), whose maps are staged: R0 + ln + i stride for
// each of the workgroup's rows ln.  First the groups of four whole pixels on
// one side of the centre, each thread down its columns; then the group across
// the centre and the one at the row's ragged end, if any, a thread per row.
template <int C, int BPS, int KIND, bool WRITE, bool STATS, bool VB>
__device__ inline void piece_rows(const Geo& g, const Bufs& b, const DevCam& cam, int k, __amdgpu_buffer_rsrc_t rin,
                                  __amdgpu_buffer_rsrc_t rout, int R0, int step, int p0, int p1, int j0,
                                  ApplyLds& L, Sums16& sums, int tid) {
  constexpr int NW = C * BPS;
  constexpr int kU = rows_in_flight(KIND, C, STATS);
  const int cols = cam.ap_cols, lanes = cam.ap_lanes;
  const int W = cam.width, half = cam.half, pitch = (int)cam.pitch;
  const int ngroups = (W + 3) >> 2;
  const int hrep = tid & (kRep - 1);
  const int shift = cam.bit_depth - 8;
  const uint32_t maxv = (1u << cam.bit_depth) - 1u;
  const uint16_t* wrow = b.weights + (int64_t)k * g.w_max;
  auto weights_of = [&](int col0, int npx, uint32_t (&wp)[4]) {
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const uint32_t w = WRITE && p < npx ? (uint32_t)wrow[col0 + p] : 0u;
      wp[p] = (256u - w) | (w << 16);
    }
  };
  const int ln = tid / cols;
  int first = R0 + ln;                    // this thread's first row of the piece
  if (first < p0) first += (p0 - first + step - 1) / step * step;
  if (ln < lanes && first < p1) {         // so rows are in [p0, p1), inside a staged entry
    // A step takes at least `skip` blocks on.
    const int skip = (int)((uint32_t)step * (uint32_t)g.n_blocks / (uint32_t)cam.height);
    for (int grp = tid - ln * cols; grp < ngroups; grp += cols) {
      const int col0 = grp * 4;
      const int side = col0 >= half ? 1 : 0;
      if (col0 + 4 > W || (col0 < half && col0 + 3 >= half)) continue;
      const int cbyte = col0 * NW;
      uint32_t wp[4];
      weights_of(col0, 4, wp);
      // Staged entry of the row, rows taken in turn (every step-th): whether it
      // is another one than before.
      int e = VB ? (first - p0) / step * lanes + ln - lanes : -1;
      auto next_entry = [&](int row) {
        if (VB) {
          e += lanes;
          return true;
        }
        const int was = e;
        e = e < 0 ? row_block(row, cam.height, g.n_blocks) - j0 : e + skip;
        while (row >= L.end[e]) ++e;      // at most the block after, and blocks without rows
        return e != was;
      };
      SideMap<C, KIND> m;
      for (int row = first; row < p1; row += kU * step) {
        uint32_t d[kU][NW];
#pragma unroll
        for (int u = 0; u < kU; ++u)
          if (row + u * step < p1) load_group<NW>(rin, (row + u * step) * pitch + cbyte, d[u]);
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          if (row + u * step < p1) {
            if (WRITE && next_entry(row + u * step)) m.read(L, e, side);
            uint32_t o[NW];
            one_group<C, BPS, WRITE, STATS>(d[u], o, 4, m, wp, L, hrep, shift, maxv, sums);
            if (WRITE) store_group<NW>(rout, (row + u * step) * pitch + cbyte, o);
          }
        }
      }
    }
  }
  const bool across = (half & 3) != 0, ragged = (W & 3) != 0;
  if (!across && !ragged) return;
  const int gc = half >> 2, gr = ngroups - 1;
  const int per = across && ragged && gc != gr ? 2 : 1;      // such groups of a row
  const int t0 = (p0 - R0) / step;                           // turns of the workgroup's rows in the piece
  const int turns = (p1 - R0 + step - 1) / step - t0;
#pragma unroll 1
  for (int i = tid; i < turns * lanes * per; i += kApplyThreads) {
    const int ri = i / per, turn = ri / lanes, l = ri - turn * lanes;
    const int row = R0 + (t0 + turn) * step + l;
    if (row < p0 || row >= p1) continue;
    const int grp = i - ri * per == 0 && across ? gc : gr;
    const int col0 = grp * 4, npx = min(4, W - col0);
    const int side = col0 >= half ? 1 : 0;
    const int off = row * pitch + col0 * NW;
    uint32_t d[NW], o[NW], wp[4];
    load_part<NW>(rin, off, npx * NW, d);
    weights_of(col0, npx, wp);
    SideMap<C, KIND> m;
    const int e = VB ? ri : row_block(row, cam.height, g.n_blocks) - j0;
    if (WRITE) m.read(L, e, side);
    one_group<C, BPS, WRITE, STATS>(d, o, npx, m, wp, L, hrep, shift, maxv, sums);
    if (WRITE) {
      if (col0 < half && col0 + 3 >= half) {
        // The pixels from half on, again with the right side's maps.
        uint32_t q[NW];
        m.read(L, e, 1);
        one_group<C, BPS, WRITE, false>(d, q, npx, m, wp, L, hrep, shift, maxv, sums);
        const int keep = (half - col0) * NW;                 // bytes of the left side's pixels
#pragma unroll
        for (int n = 0; n < NW; ++n) {
          const int kept = min(max(keep - 4 * n, 0), 4);
          const uint32_t mask = kept == 4 ? ~0u : (1u << (8 * kept)) - 1u;
          o[n] = (o[n] & mask) | (q[n] & ~mask);
        }
      }
      store_part<NW>(rout, off, npx * NW, o);
    }
  }
}

// Adds the run's LDS histogram of camera k (replicas summed) and its (n, S1,
// S2) - linear in the histogram for 8-bit samples, the threads' sums for
// 16-bit ones - to the camera's whole-frame statistics.
template <int C, int BPS>
__device__ inline void flush_whole(const Bufs& b, int k, ApplyLds& L, const Sums16& sums, int tid) {
  const int lane = tid % kWave;
  auto add = [&](int i, unsigned long long s) {
    if (lane == 0)
      __hip_atomic_fetch_add(&L.sums[i], s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  __syncthreads();
  uint32_t* gh = b.whole_hist + (int64_t)k * kCS * kNB;
  for (int i = tid; i < C * kNB; i += kApplyThreads) {    // whole waves, one channel each
    const u32x4* h4 = reinterpret_cast<const u32x4*>(&L.hist[i * kRep]);
    uint32_t h = 0;
#pragma unroll
    for (int q = 0; q < kRep / 4; ++q) {
      const u32x4 v = h4[q];
      h += v.x + v.y + v.z + v.w;
    }
    if (h) atomicAdd(&gh[i], h);
    const int c = i / kNB;
    const unsigned long long x = (unsigned long long)(i % kNB);
    add(c * 3, wave_sum_u64(h));
    if (BPS == 1) {
      add(c * 3 + 1, wave_sum_u64(h * x));
      add(c * 3 + 2, wave_sum_u64(h * x * x));
    }
  }
  if (BPS == 2) {
    add(1, wave_sum_u64(sums.s1));
    add(2, wave_sum_u64(sums.s2));
  }
  __syncthreads();
  if (tid < 3 * C && L.sums[tid]) atomicAdd((unsigned long long*)&b.whole_sums[(int64_t)k * 9 + tid], L.sums[tid]);
}

// The run's rows R0 + ln + i stride (ln < ap_lanes) below R1 of camera k, of C
// channels of BPS bytes (see RowRun).  CROSS: the 3x3 maps q3 in place of the affine ones.
template <int C, int BPS, bool WRITE, bool STATS, bool VB, bool CROSS, class FP>
__device__ __attribute__((always_inline)) inline void apply_rows(const Geo& g, const FP& fp, const Bufs& b,
                                                                 const int64_t* q3, const DevCam& cam, int k,
                                                                 const RowRun& run, ApplyLds& L) {
  // The thread's index as a value of its own in every camera and form: else what
  // follows from it is worked out for all of them ahead of the loop over cameras,
  // kept in registers and, at 96, spilled.
  int tid = threadIdx.x;
  asm("" : "+v"(tid));
  const int H = cam.height, nb = g.n_blocks;
  const int R0 = run.row0, R1 = run.row1, stride = run.stride;
  if (STATS) {
    const u32x4 zero = {0, 0, 0, 0};
    for (int i = tid; i < C * kNB * kRep / 4; i += kApplyThreads) reinterpret_cast<u32x4*>(L.hist)[i] = zero;
    if (tid < 9) L.sums[tid] = 0;
  }
  const __amdgpu_buffer_rsrc_t rin = frame_rsrc(fp.in[k], cam);
  __amdgpu_buffer_rsrc_t rout = rin;
  if (WRITE) rout = frame_rsrc(fp.out[k], cam);
  Sums16 sums = {0, 0};
  if constexpr (!WRITE) {
    __syncthreads();
    piece_rows<C, BPS, kMapDirect, WRITE, STATS, false>(g, b, cam, k, rin, rout, R0, stride, R0, R1, 0, L, sums, tid);
  } else {
    // The run in pieces whose maps fit the staging area.  Where a map is too
    // large for the fast form, the entries before it are taken first, then
    // its own block (or, blended, its turn of the workgroup's rows) in the exact
    // form.
    constexpr int kFast = CROSS ? kMapCross : BPS == 2 ? kMapWide : VB || STATS ? kMapDirect : kMapTable;
    constexpr int kExact = CROSS ? kMapCrossWide : VB ? kMapWide : kMapTable;
    constexpr bool kChecked = kFast == kMapDirect || kFast == kMapCross;
    constexpr int kCap = MapEntry<kFast, C>::kCap;
    const int per = VB ? cam.ap_lanes : 1;                // entries of a block or turn
    const int je = VB ? 0 : row_block(R1 - 1, H, nb);
#pragma unroll 1
    for (int p0 = R0, p1; p0 < R1; p0 = p1) {
      const int j0 = VB ? 0 : row_block(p0, H, nb);
      // Blocks (VB: turns) at hand, and the end of the rows of the first n of them.
      int n = VB ? min(max(1, kCap / per), (R1 - p0 + stride - 1) / stride) : min(kCap, je - j0 + 1);
      auto end = [&](int m) { return min(R1, VB ? p0 + m * stride : block_row(j0 + m, H, nb)); };
      if (p0 != R0) __syncthreads();      // the previous piece's rows are done with the maps
      const int good = stage_maps<C, BPS, kFast, VB>(g, b, q3, cam, k, p0, stride, j0, n * per, L, tid) / per;
      if (!kChecked || good > 0) {
        p1 = end(kChecked ? good : n);
        piece_rows<C, BPS, kFast, WRITE, STATS, VB>(g, b, cam, k, rin, rout, R0, stride, p0, p1, j0, L, sums, tid);
      } else if constexpr (kChecked) {
        __syncthreads();
        (void)stage_maps<C, BPS, kExact, VB>(g, b, q3, cam, k, p0, stride, j0, per, L, tid);
        p1 = end(1);
        piece_rows<C, BPS, kExact, WRITE, STATS, VB>(g, b, cam, k, rin, rout, R0, stride, p0, p1, j0, L, sums, tid);
      }
    }
  }
  if (STATS) flush_whole<C, BPS>(b, k, L, sums, tid);
}

// Sums of v over the lanes up to and including the own one (all lanes active).
__device__ inline unsigned long long wave_prefix_u64(unsigned long long v) {
  v += dpp_u64<0x111>(v);          // row_shr:1
  v += dpp_u64<0x112>(v);          // row_shr:2
  v += dpp_u64<0x114>(v);          // row_shr:4
  v += dpp_u64<0x118>(v);          // row_shr:8
  v += dpp_u64<0x142, 0xa>(v);     // row_bcast:15 into rows 1 and 3
  v += dpp_u64<0x143, 0xc>(v);     // row_bcast:31 into rows 2 and 3
  return v;
}

// Run w of the default split over the active cameras of a larger rig, worked out
// here, a lane per camera, as split_shares does: the context's table shares the
// workgroups among all cameras and would leave a few of them with a few.  (The
// shares as a kernel argument of 130 bytes cost every launch of the library 0.1
// us.)  rt_frameset_batch, apply us, table and this: one 1920x1080 camera of 32
// 45.9 and 15.5 (28.5 with one workgroup per tile), one 1280x720 of 60 38.4 and
// 10.9 (26.4), seven 1920x1080 of 14 36.7 and 26.7 (37.9).
__device__ inline WgRun subset_run(const Geo& g, int w) {
  static_assert(RT_MAX_CAMS <= kWave, "a lane per camera");
  const int lane = threadIdx.x % kWave;
  int64_t bytes = 0;
  int32_t steps = 0, height = 0, lanes = 1;
  if (lane < g.n_cams && cam_active(g, lane)) {
    const DevCam& c = g.cams[lane];
    height = c.height;
    lanes = c.ap_lanes;
    bytes = (int64_t)height * c.row_bytes;
    steps = (height + lanes - 1) / lanes;
  }
  const int64_t upto = (int64_t)wave_prefix_u64(bytes);
  const int64_t all = (int64_t)wave_sum_u64(bytes), all_steps = (int64_t)wave_sum_u64(steps);
  const int share = steps ? camera_share(split_total(all_steps) - __popcll(g.active), upto - bytes, bytes, all, steps) : 0;
  const int end = (int)wave_prefix_u64(share);
  const int k = __popcll(__builtin_amdgcn_ballot_w64(end <= w));   // (the lanes beyond the last camera hold the total)
  const int m = __builtin_amdgcn_readlane(share, k), i = w - (__builtin_amdgcn_readlane(end, k) - m);
  height = __builtin_amdgcn_readlane(height, k);
  lanes = __builtin_amdgcn_readlane(lanes, k);
  const bool interleave = runs_interleave(__builtin_amdgcn_readlane(steps, k), m, g.n_blocks);
  const RowRun r = row_run(height, lanes, i, m, interleave), t = row_run(height, lanes, i, m, false);
  return WgRun{k, r.row0, k, r.row1, r.stride, t.row0, t.row1};
}

// Workgroup w's run: its rows of every camera it takes.
template <bool WRITE, bool STATS, bool VB, bool CROSS, class FP>
__device__ __attribute__((always_inline)) inline void apply_run(const Geo& g, const FP& fp, const Bufs& b,
                                                                const int64_t* q3, int w, ApplyLds& L) {
  const WgRun run = g.runs ? uniform_run(g, w) : subset_run(g, w);
  for (int k = run.cam0; k <= run.cam1; ++k) {
    if (!cam_active(g, k)) continue;              // uniform over the workgroup
    const DevCam cam = uniform_cam(g, k);
    RowRun r = {k == run.cam0 ? run.row0 : 0, k == run.cam1 ? run.row1 : cam.height, cam.ap_lanes};
    if (run.stride) {
      if (WRITE && !STATS && !VB && !CROSS && cam.bps == 1) r = RowRun{run.trow0, run.trow1, cam.ap_lanes};
      else r.stride = run.stride;
    }
    if (r.row0 >= r.row1) continue;
    if constexpr (CROSS) {
      apply_rows<3, 1, WRITE, STATS, VB, true>(g, fp, b, q3, cam, k, r, L);
    } else if (cam.bps == 2) {
      apply_rows<1, 2, WRITE, STATS, VB, false>(g, fp, b, q3, cam, k, r, L);
    } else if (cam.channels == 3) {
      apply_rows<3, 1, WRITE, STATS, VB, false>(g, fp, b, q3, cam, k, r, L);
    } else {
      apply_rows<1, 1, WRITE, STATS, VB, false>(g, fp, b, q3, cam, k, r, L);
    }
    if (k < run.cam1) __syncthreads();
  }
}

}  // namespace rc
