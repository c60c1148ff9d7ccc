// Band statistics of section 3.1 as device functions: the histogram and sums
// of one (camera, side, block) unit, optionally with the sums of its pixels
// that do not move against the previous frame (object removal) or with its
// cross sums over the channels; and the clearing of the whole-frame
// statistics that the apply pass accumulates.
#pragma once

#include <type_traits>

#include "dev_common.h"

namespace rc {

// Previous frames of a launch (device pointers; all NULL: nothing moves).
struct PrevPtrs {
  const uint8_t* in[RT_MAX_CAMS];
};

// Object-removal arguments of a launch.
struct Removal {
  uint64_t* kept_sums;   // [K][2][NB][3][3] (n, S1, S2) of the kept pixels
  uint8_t* method;       // [K][2][NB] method taken by each unit (may be NULL)
  int32_t tau;           // threshold in 8-bit units
  int32_t has_prev;      // 0: no previous frames, every pixel is kept
  double min_kept;       // least kept fraction of both bands for the removal fit
};

// What a band pass gathers beside the histogram and (n, S1, S2).
enum { kBandPlain, kBandMotion, kBandCross };

struct BandArgs {
  const PrevPtrs* pp;        // kBandMotion
  const Removal* rm;
  uint64_t* cross;           // kBandCross: [unit][3]
};

constexpr int kPartMax = 7;    // sums a thread accumulates itself
constexpr int kBandWaves = 4;  // most waves of a band pass

// REP: histogram replicas, interleaved bin by bin, lane l updating replica l %
// REP.  A wave's lanes hold one channel of a few neighbouring rows, so many of
// them meet in one bin, and atomics on one LDS word go one after the other: with
// a single histogram they were 9 of the seam kernel's 14 us on the 14x1920x1080
// rig.  Its time there by replicas: 1 13.6 us, 4 8.2, 8 7.6, 16 8.2.
template <int REP>
struct BandLds {
  static constexpr int kRep = REP;
  static_assert(REP >= 4 && (REP & (REP - 1)) == 0, "replicas, summed four at a time");
  alignas(16) uint32_t hist[kCS * kNB * REP];
  unsigned long long part[kBandWaves][kPartMax];
};
constexpr int kBandRep = 8;

// Barriers (__syncthreads) that band_unit passes, on every path.
constexpr int kBandBarriers = 3;

// Four pixels of a band row as loaded: the dwords that hold them, the first
// starting at the aligned byte at or before the group, and the third byte of
// a last dword that is cut by the row's end after three bytes.
template <int ND>
struct BandGroup {
  uint32_t d[ND + 1];
  uint32_t x;
};

// Loads the nb bytes at byte offset o of the row at rowoff; SHIFTED: any o and
// nb (no byte beyond the row's end is touched), else o is a multiple of 4 and
// nb = 4 ND.
template <int ND, bool SHIFTED>
__device__ inline void load_band(__amdgpu_buffer_rsrc_t r, int rowoff, int o, int nb, int row_bytes,
                                 BandGroup<ND>& v) {
  if constexpr (!SHIFTED) {
    if constexpr (ND == 3) {
      typedef unsigned int u32x3 __attribute__((ext_vector_type(3)));
      const u32x3 t = __builtin_amdgcn_raw_buffer_load_b96(r, rowoff + o, 0, 0);
      v.d[0] = t.x; v.d[1] = t.y; v.d[2] = t.z;
    } else if constexpr (ND == 2) {
      typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
      const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(r, rowoff + o, 0, 0);
      v.d[0] = t.x; v.d[1] = t.y;
    } else {
      v.d[0] = __builtin_amdgcn_raw_buffer_load_b32(r, rowoff + o, 0, 0);
    }
    return;
  }
  const int base = o & ~3, end = o + nb;
  v.x = 0;
#pragma unroll
  for (int i = 0; i <= ND; ++i) {
    const int at = base + 4 * i, have = row_bytes - at;
    v.d[i] = 0;
    if (at < end) {
      if (have >= 4) v.d[i] = __builtin_amdgcn_raw_buffer_load_b32(r, rowoff + at, 0, 0);
      else if (have >= 2) {
        v.d[i] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, rowoff + at, 0, 0);
        if (have == 3) v.x = (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(r, rowoff + at + 2, 0, 0);
      } else {
        v.d[i] = (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(r, rowoff + at, 0, 0);
      }
    }
  }
}

// The group's ND dwords, its first byte in the lowest byte of w[0].
template <int ND, bool SHIFTED>
__device__ inline void band_dwords(const BandGroup<ND>& v, int o, int row_bytes, uint32_t (&w)[ND]) {
  if constexpr (!SHIFTED) {
#pragma unroll
    for (int i = 0; i < ND; ++i) w[i] = v.d[i];
  } else {
    const int cut = row_bytes - (o & ~3);          // the third byte belongs to the dword that holds offset cut - 1
    uint32_t d[ND + 1];
#pragma unroll
    for (int i = 0; i <= ND; ++i) d[i] = cut == 4 * i + 3 ? v.d[i] | (v.x << 16) : v.d[i];
#pragma unroll
    for (int i = 0; i < ND; ++i) w[i] = __builtin_amdgcn_alignbyte(d[i + 1], d[i], (uint32_t)(o & 3));
  }
}

// Sample i (0 .. 4 C - 1 in pixel-major order) of a group of 4 pixels.
template <int BPS>
__device__ inline uint32_t group_sample(const uint32_t* w, int i) {
  if (BPS == 1) return (w[i >> 2] >> (8 * (i & 3))) & 0xffu;
  return (w[i >> 1] >> (16 * (i & 1))) & 0xffffu;
}

// Band statistics of unit (k, s, j) by HT threads (whole waves; tid: the
// thread's index among them): histogram and exact (n, S1, S2) of the band's
// samples into the caller's buffers.  The threads walk the band in groups of 4
// pixels, kB groups per thread in flight; the first ones are loaded while the
// histogram is cleared.  8-bit sums follow from the histogram, one wave per
// channel; 16-bit ones, the kept sums (kBandMotion) and the cross sums
// (kBandCross) are accumulated by the threads.  sums / extra (LDS, may be
// NULL) also receive the nine sums and the nine kept or three cross sums.
template <int C, int BPS, int HT, int WHAT, bool SHIFTED, class Lds>
__device__ __attribute__((always_inline)) inline void band_pass(const Geo& g, const FramePtrs& fp, const Bufs& b,
                                                                const BandArgs& a, const DevCam& cam, int k, int s,
                                                                int j, Lds& L, uint64_t* sums, uint64_t* extra,
                                                                int tid) {
  constexpr int ND = C * BPS;                 // dwords of a 4-pixel group
  constexpr int kRep = Lds::kRep;
  constexpr bool kMotion = WHAT == kBandMotion, kCross = WHAT == kBandCross;
  constexpr int kB = HT >= 256 ? 3 : kMotion ? 3 : 5;
  constexpr int kParts = kMotion ? 1 + 2 * C : kCross ? 3 : 0;
  constexpr int kPart16 = kParts;             // first of the two 16-bit sums
  constexpr int kAll = kParts + (BPS == 2 ? 2 : 0);
  static_assert(kAll <= kPartMax && HT / kWave <= kBandWaves, "partial sums");
  const int nb = g.n_blocks;
  const int r0 = (int)((uint32_t)j * (uint32_t)cam.height / (uint32_t)nb);
  const int r1 = (int)((uint32_t)(j + 1) * (uint32_t)cam.height / (uint32_t)nb);
  const int band = cam.band, rows = r1 - r0;
  const int c0 = s == 0 ? 0 : cam.width - band;
  const int ng = (band + 3) >> 2;             // groups per band row
  const int shift = cam.bit_depth - 8;
  const int pitch = (int)cam.pitch;
  const __amdgpu_buffer_rsrc_t rin = frame_rsrc(fp.in[k], cam);
  uint32_t thr = 0;
  bool has_prev = false;
  __amdgpu_buffer_rsrc_t rprev = rin;
  if constexpr (kMotion) {
    thr = (uint32_t)a.rm->tau << shift;
    has_prev = a.rm->has_prev != 0;
    if (has_prev) rprev = frame_rsrc(a.pp->in[k], cam);
  }
  // Walk over (row, group): HT groups on is drow rows and dq groups on.
  const int total = rows * ng;
  int row = ng ? tid / ng : 0, q = tid - row * ng;
  const int drow = ng ? HT / ng : 0, dq = HT - drow * ng;
  auto next = [&](int& rw, int& qq) {
    rw += drow;
    qq += dq;
    if (qq >= ng) { qq -= ng; ++rw; }
  };
  BandGroup<ND> v[kB], pv[kMotion ? kB : 1];
  auto fetch = [&](int rw, int qq) {
#pragma unroll
    for (int i = 0; i < kB; ++i) {
      if (rw < rows) {
        const int off = (r0 + rw) * pitch, o = (c0 + 4 * qq) * ND;
        const int n = min(4, band - 4 * qq) * ND;
        load_band<ND, SHIFTED>(rin, off, o, n, cam.row_bytes, v[i]);
        if (kMotion && has_prev) load_band<ND, SHIFTED>(rprev, off, o, n, cam.row_bytes, pv[kMotion ? i : 0]);
      }
      next(rw, qq);
    }
  };
  if (total > 0) fetch(row, q);
  {
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 zero = {0, 0, 0, 0};
    for (int i = tid; i < C * kNB * kRep / 4; i += HT) reinterpret_cast<u32x4*>(L.hist)[i] = zero;
  }
  __syncthreads();

  const int rep = tid & (kRep - 1);
  unsigned long long a1 = 0, a2 = 0;          // 16-bit sums
  uint32_t kn = 0;
  unsigned long long k1[C], k2[C];            // kept sums; cross: k2 the three products
#pragma unroll
  for (int c = 0; c < C; ++c) k1[c] = k2[c] = 0;
  if (total > 0) {
    for (int it = tid; it < total; it += kB * HT) {
      if (it != tid) fetch(row, q);
#pragma unroll
      for (int i = 0; i < kB; ++i) {
        if (row < rows) {
          const int o = (c0 + 4 * q) * ND;
          uint32_t w[ND], p[ND];
          band_dwords<ND, SHIFTED>(v[i], o, cam.row_bytes, w);
          if (kMotion && has_prev) band_dwords<ND, SHIFTED>(pv[kMotion ? i : 0], o, cam.row_bytes, p);
          const int npx = SHIFTED ? min(4, band - 4 * q) : 4;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (e < npx) {
              uint32_t x[C];
              bool moving = false;
#pragma unroll
              for (int c = 0; c < C; ++c) {
                x[c] = group_sample<BPS>(w, e * C + c);
                if (kMotion && has_prev) {
                  const uint32_t y = group_sample<BPS>(p, e * C + c);
                  moving = moving || (x[c] > y ? x[c] - y : y - x[c]) > thr;
                }
                uint32_t bin = x[c];
                if (BPS == 2) {
                  bin >>= shift;
                  bin = bin > 255u ? 255u : bin;
                  a1 += x[c];
                  a2 += (unsigned long long)x[c] * x[c];
                }
                __hip_atomic_fetch_add(&L.hist[(c * kNB + bin) * kRep + rep], 1u, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
              }
              if (kMotion && !moving) {
                ++kn;
#pragma unroll
                for (int c = 0; c < C; ++c) {
                  k1[c] += x[c];
                  k2[c] += (unsigned long long)x[c] * x[c];
                }
              }
              if constexpr (kCross) {
                k2[0] += x[0] * x[1];
                k2[1] += x[0] * x[2];
                k2[2] += x[1] * x[2];
              }
            }
          }
        }
        next(row, q);
      }
    }
  }
  const int wave = tid / kWave, lane = tid % kWave;
  if constexpr (kAll > 0) {
    // Partial sums: kept n, S1 and S2 per channel (or the cross sums), then
    // the 16-bit S1 and S2.
    auto part = [&](int i, unsigned long long t) {
      t = wave_sum_u64(t);
      if (lane == 0) L.part[wave][i] = t;
    };
    if constexpr (kMotion) {
      part(0, kn);
#pragma unroll
      for (int c = 0; c < C; ++c) {
        part(1 + c, k1[c]);
        part(1 + C + c, k2[c]);
      }
    }
    if constexpr (kCross) {
#pragma unroll
      for (int c = 0; c < 3; ++c) part(c, k2[c < C ? c : 0]);
    }
    if constexpr (BPS == 2) {
      part(kPart16, a1);
      part(kPart16 + 1, a2);
    }
  }
  __syncthreads();

  auto total_of = [&](int i) {
    unsigned long long t = 0;
#pragma unroll
    for (int w = 0; w < HT / kWave; ++w) t += L.part[w][i];
    return t;
  };
  const int64_t u0 = unit_index(k, s, j, 0, nb);
  // One wave per channel: the histogram written out, lane l holding bins l, l +
  // 64, l + 128 and l + 192, and its sums.
  for (int c = wave; c < kCS; c += HT / kWave) {
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    unsigned long long s1 = 0, s2 = 0;
#pragma unroll
    for (int i = 0; i < kNB / kWave; ++i) {
      const int bin = i * kWave + lane;
      uint32_t h = 0;
      if (c < C) {
#pragma unroll
        for (int q = 0; q < kRep / 4; ++q) {
          const u32x4 t = reinterpret_cast<const u32x4*>(L.hist + (c * kNB + bin) * kRep)[q];
          h += t.x + t.y + t.z + t.w;
        }
      }
      b.band_hist[(u0 + c) * kNB + bin] = h;
      const unsigned long long t1 = (unsigned long long)h * (unsigned)bin;
      s1 += t1;
      s2 += t1 * (unsigned)bin;
    }
    if (BPS == 2) {
      s1 = s2 = 0;
      if (c < C) {
        s1 = total_of(kPart16);
        s2 = total_of(kPart16 + 1);
      }
    } else if (c < C) {
      s1 = wave_sum_u64(s1);
      s2 = wave_sum_u64(s2);
    }
    if (lane < 3) {
      const unsigned long long n = c < C ? (unsigned long long)rows * (unsigned long long)band : 0ull;
      const unsigned long long t = lane == 0 ? n : (lane == 1 ? s1 : s2);
      b.band_sums[(u0 + c) * 3 + lane] = t;
      if (sums) sums[c * 3 + lane] = t;
    }
  }
  if constexpr (kMotion) {
    // Kept sums per channel slot, n repeated for every channel of the camera.
    if (tid < 9) {
      const int c = tid / 3, m = tid - 3 * (tid / 3);
      const unsigned long long t = c >= C ? 0ull : total_of(m == 0 ? 0 : (m == 1 ? 1 + c : 1 + C + c));
      a.rm->kept_sums[u0 * 3 + tid] = t;
      if (extra) extra[tid] = t;
    }
  }
  if constexpr (kCross) {
    if (tid < 3) {
      const unsigned long long t = total_of(tid);
      a.cross[u0 + tid] = t;
      if (extra) extra[tid] = t;
    }
  }
  __syncthreads();
}

// Band statistics of unit (camera, side, block) = `unit` by HT threads (see
// band_pass); kBandCross takes RGB8 cameras only.
template <int HT, int WHAT, class Lds>
__device__ __attribute__((always_inline)) inline void band_unit(const Geo& g, const FramePtrs& fp, const Bufs& b,
                                                                const BandArgs& a, int unit, Lds& L,
                                                                uint64_t* sums, uint64_t* extra, int tid) {
  const int nb = g.n_blocks;
  const int k = unit / (2 * nb);
  const int s = (unit / nb) & 1;
  const int j = unit % nb;
  const DevCam cam = uniform_cam(g, k);
  // Whole groups of four pixels on dword boundaries.
  const int start = (s == 0 ? 0 : cam.width - cam.band) * cam.channels * cam.bps;
  const bool whole = (cam.band & 3) == 0 && (start & 3) == 0;
  auto pass = [&](auto c, auto bps) {
    if (whole) band_pass<decltype(c)::value, decltype(bps)::value, HT, WHAT, false>(g, fp, b, a, cam, k, s, j, L, sums, extra, tid);
    else band_pass<decltype(c)::value, decltype(bps)::value, HT, WHAT, true>(g, fp, b, a, cam, k, s, j, L, sums, extra, tid);
  };
  using one = std::integral_constant<int, 1>;
  using two = std::integral_constant<int, 2>;
  using three = std::integral_constant<int, 3>;
  if constexpr (WHAT == kBandCross) {
    pass(three{}, one{});
  } else {
    if (cam.bps == 2) pass(one{}, two{});
    else if (cam.channels == 3) pass(three{}, one{});
    else pass(one{}, one{});
  }
}

// The seam block (camera k, block j) = bid: its units are u[0], the right band
// of camera k; the band that one faces, if any; and at the start of an open
// ring camera k's left band, which faces nothing.  Over the rig every unit is
// in exactly one seam block, and only units 0 and 1 of a seam with `faces` set
// face each other.
struct Seam {
  int k, j, n;
  int u[3];
  bool faces;
};

__device__ inline Seam seam_of(const Geo& g, const DevCam& cam, int k, int j) {
  const int nb = g.n_blocks;
  Seam m;
  m.k = k;
  m.j = j;
  m.faces = cam.face_cam[1] >= 0;
  m.u[0] = (k * 2 + 1) * nb + j;
  m.u[1] = m.u[2] = 0;
  m.n = 1;
  if (m.faces) m.u[m.n++] = (cam.face_cam[1] * 2 + cam.face_side[1]) * nb + j;
  if (cam.face_cam[0] < 0) {
    (m.n == 1 ? m.u[1] : m.u[2]) = k * 2 * nb + j;
    ++m.n;
  }
  return m;
}

// Band statistics of a seam's units by a workgroup of NT threads, two units at
// a time, each by one half of it; unit i's sums (and its kept or cross sums)
// are left in sums[i] (extra[i]).
template <int NT, int WHAT, class Lds>
__device__ __attribute__((always_inline)) inline void seam_bands(const Geo& g, const FramePtrs& fp, const Bufs& b,
                                                                 const BandArgs& a, const Seam& m, Lds (&L)[2],
                                                                 uint64_t (&sums)[3][9], uint64_t (&extra)[3][9]) {
  constexpr int HT = NT / 2;
  static_assert(HT % kWave == 0, "whole waves");
  const int tid = threadIdx.x;
  const int half = uniform((int32_t)(tid / HT)), ltid = tid - half * HT;
#pragma unroll 1
  for (int p = 0; p < m.n; p += 2) {
    const int i = p + half;
    if (i < m.n) {
      band_unit<HT, WHAT>(g, fp, b, a, i == 0 ? m.u[0] : (i == 1 ? m.u[1] : m.u[2]), L[half], sums[i], extra[i], ltid);
    } else {
      for (int w = 0; w < kBandBarriers; ++w) __syncthreads();
    }
  }
}

// Zero the whole-frame histogram and sums of every active camera (grid-stride).
__device__ inline void zero_whole(const Geo& g, const Bufs& b, int thread, int nthreads) {
  const int nh = g.n_cams * kCS * kNB;
  for (int i = thread; i < nh; i += nthreads)
    if (cam_active(g, i / (kCS * kNB))) b.whole_hist[i] = 0u;
  for (int i = thread; i < g.n_cams * 9; i += nthreads)
    if (cam_active(g, i / 9)) b.whole_sums[i] = 0ull;
}

}  // namespace rc
