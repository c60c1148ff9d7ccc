// Estimate and table kernels of section 3.1: one thread per (camera, side,
// block, channel) for the affine fit, one workgroup per (camera, side, block)
// for the tables, one thread per column for the blend weights; the
// look-ahead frame-set kernel (the apply of one frame-set in the same launch
// as the seam estimate of the next).
#include "dev_apply.h"
#include "dev_estimate.h"
#include "dev_stats.h"
#include "rt_ahead_internal.h"

namespace rc {

__global__ __launch_bounds__(kThreads) void k_estimate(Geo g, Bufs b) {
  const int u = blockIdx.x * blockDim.x + threadIdx.x;
  if (u < g.n_cams * 2 * g.n_blocks * kCS && cam_active(g, u / (2 * g.n_blocks * kCS))) estimate_unit(g, b, u);
}

// The quantile fit of every unit (RT_FIT_QUANTILE), one wave per (camera,
// side, block, channel) unit: the wave gathers the quantiles of the unit's
// band and of the band it faces from the band histograms, its first lane fits
// and updates the state.
__global__ __launch_bounds__(kThreads) void k_estimate_quantile(Geo g, Bufs b) {
  __shared__ uint32_t cum[kThreads / kWave][2 * kNB];
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int u = uniform((int32_t)(blockIdx.x * (kThreads / kWave) + wave));
  const int nb = g.n_blocks;
  if (u >= g.n_cams * 2 * nb * kCS) return;    // the whole wave
  const int c = u % kCS, j = (u / kCS) % nb, s = (u / (kCS * nb)) & 1, k = u / (kCS * nb * 2);
  if (!cam_active(g, k)) return;
  const DevCam cam = uniform_cam(g, k);
  const int fc = cam.face_cam[s];
  const int64_t uf = fc < 0 ? -1 : unit_index(fc, cam.face_side[s], j, c, nb);
  const uint64_t n_own = b.band_sums[(int64_t)u * 3];
  const uint64_t n_fac = uf < 0 ? 0 : b.band_sums[uf * 3];
  QSums q = {0, 0, 0, 0, 0};
  if (c < cam.channels && uf >= 0 && n_own != 0 && n_fac != 0)
    q = wave_quantile_sums(b.band_hist + (int64_t)u * kNB, b.band_hist + uf * kNB, cam.bit_depth - 8 > 0 ? cam.bit_depth - 8 : 0,
                           cum[wave], lane);
  if (lane == 0) {
    double a, bb;
    const int st = fit_quantile(g, cam.channels, c, uf >= 0, n_own, n_fac, q, true, a, bb);
    temporal_update(g, b.params, b.valid, u, st, a, bb);
  }
}

__global__ __launch_bounds__(kThreads) void k_build_lut(Geo g, Bufs b) {
  if (!cam_active(g, blockIdx.x / (2 * g.n_blocks))) return;
  unit_tables(g, b, blockIdx.x, threadIdx.x);
}

__global__ __launch_bounds__(kThreads) void k_weights(Geo g, Bufs b) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)g.n_cams * g.w_max) return;
  const int k = (int)(i / g.w_max);
  const int col = (int)(i - (int64_t)k * g.w_max);
  if (cam_active(g, k)) b.weights[i] = (uint16_t)blend_weight(g.cams[k].width, col);
}

constexpr int kBesideRep = 4;   // histogram replicas beside applies

// Band statistics, estimate and tables of a frame-set in one launch, one
// workgroup of NT threads per seam block (see Seam).  A unit's estimate needs
// only its own band and the one it faces, so after the statistics of its
// bands the workgroup fits those units and builds their tables with no other
// workgroup involved.  Same results as k_band_stats, k_estimate, k_build_lut
// and k_weights in sequence (the whole-frame statistics that the frame-set's
// apply pass accumulates are cleared here too, when given).  WHAT ==
// kBandMotion: the band passes also sum the pixels that do not move against
// the previous frames, and each unit takes the object-removal fit or the
// smoothing fallback (removal_step), as k_motion_stats and k_estimate_removal
// would.
//
// Bound by its chain of dependent steps, not by bytes (2.9 MB of bands per
// 14x1920x1080 frame-set).  So both bands are gathered side by side, each by
// half of the workgroup with all of its loads in flight at once, one wave per
// channel sums a histogram, the fixed-point maps pass through LDS and the
// tables are built four entries per thread.  Measured on MI355X against the
// bands one after the other (us): 17.6 -> 13.6 on that rig, and 7.6 with the
// histogram in replicas (see BandLds); with object removal, whose groups were
// loaded one at a time, 38.4 -> 15.5 -> 11.0.
template <int REP>
struct SeamLds {
  BandLds<REP> band[2];
  uint64_t sums[3][9];     // (n, S1, S2) per channel of the units taken
  uint64_t extra[3][9];    // the same over their kept pixels
  int64_t q[3][kCS][2];    // their Q16 maps after the fit
};

template <int NT, int WHAT, bool QFIT, class Lds>
__device__ __attribute__((always_inline)) inline void band_estimate_body(const Geo& g, const FramePtrs& fp,
                                                                         const BandArgs& a, const Bufs& b, Lds& L,
                                                                         int bid, int nblk) {
  constexpr bool kMotion = WHAT == kBandMotion;
  static_assert(!(kMotion && QFIT), "object removal keeps only the moments of the kept pixels");
  // This kernel's chain of dependent steps is what the next apply waits
  // for; its waves take issue priority over the apply waves they share
  // compute units with (measured on MI355X: 628 -> 674 GPix/s in the
  // pipelined frame-set loop).
  __builtin_amdgcn_s_setprio(3);
  // QFIT: the quantile sums of the facing pair per channel, wave c taking
  // channel c.
  __shared__ uint32_t qcum[QFIT ? kCS : 1][QFIT ? 2 * kNB : 1];
  __shared__ QSums qs[QFIT ? kCS : 1];
  const int nb = g.n_blocks;
  const int k = bid / nb, j = bid - (bid / nb) * nb;
  const int tid = threadIdx.x;
  if (b.whole_hist) zero_whole(g, b, bid * NT + tid, nblk * NT);
  if (!cam_active(g, k)) return;
  const DevCam cam = uniform_cam(g, k);
  const Seam m = seam_of(g, cam, k, j);
  // Thread 64 t + c fits channel c of unit t: its state is read now, ahead
  // of the band passes.
  const int t = tid / kWave, c = tid % kWave;
  const bool fitter = t < m.n && c < kCS;
  const int ut = t == 0 ? m.u[0] : (t == 1 ? m.u[1] : m.u[2]);
  const int64_t u = fitter ? (int64_t)ut * kCS + c : 0;
  double p0 = 0.0, p1 = 0.0;
  uint8_t v = 0;
  if (fitter) {
    p0 = b.params[u * 2];
    p1 = b.params[u * 2 + 1];
    v = b.valid[u];
  }
  seam_bands<NT, WHAT>(g, fp, b, a, m, L.band, L.sums, L.extra);
  if constexpr (QFIT) {
    // The band histograms were written by this workgroup's band passes.
    const int wv = uniform((int32_t)(tid / kWave));
    if (m.faces && wv < cam.channels) {
      const int shift = cam.bit_depth > 8 ? cam.bit_depth - 8 : 0;
      const QSums q = wave_quantile_sums(b.band_hist + ((int64_t)m.u[0] * kCS + wv) * kNB,
                                         b.band_hist + ((int64_t)m.u[1] * kCS + wv) * kNB, shift, qcum[wv], tid % kWave);
      if (tid % kWave == 0) qs[wv] = q;
    }
    __syncthreads();
  }
  if (fitter) {
    const int other = m.faces && t < 2 ? 1 - t : -1;
    const uint64_t* own = &L.sums[t][c * 3];
    const uint64_t* fac = other >= 0 ? &L.sums[other][c * 3] : nullptr;
    // (The cameras of a ring have the same channels.)
    if constexpr (kMotion) {
      const int method = removal_method(&L.sums[t][0], other >= 0 ? &L.sums[other][0] : nullptr, &L.extra[t][0],
                                        other >= 0 ? &L.extra[other][0] : nullptr, a.rm->min_kept);
      removal_step(g, method, cam.channels, c, own, fac, &L.extra[t][c * 3],
                   other >= 0 ? &L.extra[other][c * 3] : nullptr, p0, p1, v);
      if (c == 0 && a.rm->method) a.rm->method[ut] = (uint8_t)method;
    } else {
      double fa, fb;
      int st;
      if (QFIT && fac)
        st = fit_quantile(g, cam.channels, c, true, own[0], fac[0], qs[QFIT ? c : 0], t == 0, fa, fb);
      else
        st = fit_sums(g, cam.channels, c, own, fac, fa, fb);
      temporal_step(g, st, fa, fb, p0, p1, v);
    }
    b.params[u * 2] = p0;
    b.params[u * 2 + 1] = p1;
    b.valid[u] = v;
    const int64_t A = q16_of(p0), B = q16_of(p1);
    b.q16[u * 2] = A;
    b.q16[u * 2 + 1] = B;
    L.q[t][c][0] = A;
    L.q[t][c][1] = B;
  }
  // The camera's blend weights, shared by its seam blocks.
  {
    const int w1 = (int)((int64_t)(j + 1) * g.w_max / nb);
    for (int col = (int)((int64_t)j * g.w_max / nb) + tid; col < w1; col += NT)
      b.weights[(int64_t)k * g.w_max + col] = (uint16_t)blend_weight(cam.width, col);
  }
  if (cam.bps != 1) return;
  __syncthreads();
  // Four entries of a unit's channel table per thread.
  constexpr int kQuads = kCS * kNB / 4;
  for (int i = tid; i < m.n * kQuads; i += NT) {
    const int w = i / kQuads, r = i - w * kQuads;
    const int ch = r / (kNB / 4), x = 4 * (r % (kNB / 4));
    const int unit = w == 0 ? m.u[0] : (w == 1 ? m.u[1] : m.u[2]);
    reinterpret_cast<uint32_t*>(b.lut8 + (int64_t)unit * kCS * kNB)[r] = table_quad(L.q[w][ch][0], L.q[w][ch][1], x);
  }
}

template <int NT, int REP, bool QFIT>
__global__ __launch_bounds__(NT) void k_band_estimate(Geo g, FramePtrs fp, Bufs b) {
  __shared__ SeamLds<REP> L;
  band_estimate_body<NT, kBandPlain, QFIT>(g, fp, BandArgs{}, b, L, (int)blockIdx.x, (int)gridDim.x);
}

template <int NT, int REP>
__global__ __launch_bounds__(NT) void k_band_estimate_removal(Geo g, FramePtrs fp, PrevPtrs pp, Bufs b, Removal rm) {
  __shared__ SeamLds<REP> L;
  band_estimate_body<NT, kBandMotion, false>(g, fp, BandArgs{&pp, &rm, nullptr}, b, L, (int)blockIdx.x,
                                             (int)gridDim.x);
}

// Band statistics with the kept sums, one workgroup per (camera, side, block).
__global__ __launch_bounds__(kThreads) void k_motion_stats(Geo g, FramePtrs fp, PrevPtrs pp, Bufs b, Removal rm) {
  __shared__ BandLds<kBandRep> L;
  const int unit = (int)blockIdx.x;
  if (!cam_active(g, unit / (2 * g.n_blocks))) return;
  band_unit<kThreads, kBandMotion>(g, fp, b, BandArgs{&pp, &rm, nullptr}, unit, L, nullptr, nullptr, (int)threadIdx.x);
}

// Removal fit or fallback of every (camera, side, block, channel) unit from
// the band and kept sums in the caller's layout; the channel-0 thread of a
// unit writes its method.
__global__ __launch_bounds__(kThreads) void k_estimate_removal(Geo g, Bufs b, Removal rm) {
  const int u = blockIdx.x * blockDim.x + threadIdx.x;
  if (u >= g.n_cams * 2 * g.n_blocks * kCS) return;
  const int nb = g.n_blocks;
  const int c = u % kCS, j = (u / kCS) % nb, s = (u / (kCS * nb)) & 1, k = u / (kCS * nb * 2);
  if (!cam_active(g, k)) return;
  const DevCam& cam = g.cams[k];
  const int fc = cam.face_cam[s];
  const int64_t uo = unit_index(k, s, j, 0, nb);
  const int64_t uf = fc < 0 ? -1 : unit_index(fc, cam.face_side[s], j, 0, nb);
  const uint64_t* own = b.band_sums + uo * 3;
  const uint64_t* kown = rm.kept_sums + uo * 3;
  const uint64_t* fac = uf < 0 ? nullptr : b.band_sums + uf * 3;
  const uint64_t* kfac = uf < 0 ? nullptr : rm.kept_sums + uf * 3;
  const int m = removal_method(own, fac, kown, kfac, rm.min_kept);
  double p0 = b.params[(int64_t)u * 2], p1 = b.params[(int64_t)u * 2 + 1];
  uint8_t v = b.valid[u];
  removal_step(g, m, cam.channels, c, own + c * 3, fac ? fac + c * 3 : nullptr, kown + c * 3,
               kfac ? kfac + c * 3 : nullptr, p0, p1, v);
  b.params[(int64_t)u * 2] = p0;
  b.params[(int64_t)u * 2 + 1] = p1;
  b.valid[u] = v;
  if (c == 0 && rm.method) rm.method[u / kCS] = (uint8_t)m;
}

// A frame-set of the look-ahead loop in one launch: workgroups [0, n_est)
// take the seam blocks of frame-set t + 1 (fe, be: its band statistics,
// estimate and tables, and the clearing of its whole-frame statistics, as
// k_band_estimate), the others apply frame-set t (fa, ba: with the tables an
// earlier launch built, as k_apply with statistics).  The two parts share no
// buffer and neither waits for the other; consecutive launches on a stream
// chain the estimates in order.
union AheadLds {
  ApplyLds a;
  SeamLds<kBesideRep> s;
};
template <bool VBLEND, bool QFIT>
__global__ __launch_bounds__(kApplyThreads) void k_frameset_ahead(Geo g, FramePtrs fa, Bufs ba, FramePtrs fe, Bufs be,
                                                             int n_est) {
  __shared__ AheadLds U;
  const int bid = (int)blockIdx.x;
  if (bid < n_est) {
    band_estimate_body<kApplyThreads, kBandPlain, QFIT>(g, fe, BandArgs{}, be, U.s, bid, n_est);
    return;
  }
  apply_run<true, true, VBLEND, false>(g, fa, ba, nullptr, bid - n_est, U.a);
}

hipError_t launch_frameset_ahead(const Geo& g, const FramePtrs* fa, const Bufs& ba, const FramePtrs* fe,
                                 const Bufs& be, hipStream_t st) {
  const int n_est = fe ? g.n_cams * g.n_blocks : 0, n_app = fa ? g.n_wg : 0;
  if (n_est + n_app == 0) return hipSuccess;
  const FramePtrs none = {};
  const FramePtrs& a = fa ? *fa : none;
  const FramePtrs& e = fe ? *fe : none;
  const dim3 grid(n_est + n_app), block(kApplyThreads);
  const bool q = g.fit == RT_FIT_QUANTILE;
  if (g.vblend && q) hipLaunchKernelGGL((k_frameset_ahead<true, true>), grid, block, 0, st, g, a, ba, e, be, n_est);
  else if (g.vblend) hipLaunchKernelGGL((k_frameset_ahead<true, false>), grid, block, 0, st, g, a, ba, e, be, n_est);
  else if (q) hipLaunchKernelGGL((k_frameset_ahead<false, true>), grid, block, 0, st, g, a, ba, e, be, n_est);
  else hipLaunchKernelGGL((k_frameset_ahead<false, false>), grid, block, 0, st, g, a, ba, e, be, n_est);
  return hipGetLastError();
}

// Alone on the chip the seam kernel takes the wide form, whose passes are
// shorter; beside the applies of a pipeline fewer threads and less LDS find
// room on busy compute units sooner.  14x1920x1080 rig: rt_frameset 48.8 us
// wide, 49.1 narrow with 8 replicas, 49.9 with 4; six frame-sets through the
// pipeline 240.4, 241.3 and 234.0 us; with object removal 45.5 us per frame-set
// wide and 41.0 narrow with 4, fused 44.0 and 40.5.  A two-branch graph, whose
// launches run further apart, takes 74.5 us either way and keeps the wide form.
constexpr int kNarrow = 256, kWide = 512;

hipError_t launch_band_estimate(const Geo& g, const FramePtrs& fp, const Bufs& b, hipStream_t st, bool beside) {
  const bool q = g.fit == RT_FIT_QUANTILE;
  const dim3 grid(g.n_cams * g.n_blocks), block(beside ? kNarrow : kWide);
  if (beside && q) hipLaunchKernelGGL((k_band_estimate<kNarrow, kBesideRep, true>), grid, block, 0, st, g, fp, b);
  else if (beside) hipLaunchKernelGGL((k_band_estimate<kNarrow, kBesideRep, false>), grid, block, 0, st, g, fp, b);
  else if (q) hipLaunchKernelGGL((k_band_estimate<kWide, kBandRep, true>), grid, block, 0, st, g, fp, b);
  else hipLaunchKernelGGL((k_band_estimate<kWide, kBandRep, false>), grid, block, 0, st, g, fp, b);
  return hipGetLastError();
}

const void* band_estimate_kernel(const Geo& g) {
  if (g.fit == RT_FIT_QUANTILE) return reinterpret_cast<const void*>(&k_band_estimate<kWide, kBandRep, true>);
  return reinterpret_cast<const void*>(&k_band_estimate<kWide, kBandRep, false>);
}

hipError_t launch_band_estimate_removal(const Geo& g, const FramePtrs& fp, const PrevPtrs& pp, const Bufs& b,
                                        const Removal& rm, hipStream_t st, bool beside) {
  const dim3 grid(g.n_cams * g.n_blocks);
  if (beside)
    hipLaunchKernelGGL((k_band_estimate_removal<kNarrow, kBesideRep>), grid, dim3(kNarrow), 0, st, g, fp, pp, b, rm);
  else
    hipLaunchKernelGGL((k_band_estimate_removal<kWide, kBandRep>), grid, dim3(kWide), 0, st, g, fp, pp, b, rm);
  return hipGetLastError();
}

hipError_t launch_motion_stats(const Geo& g, const FramePtrs& fp, const PrevPtrs& pp, const Bufs& b,
                               const Removal& rm, hipStream_t st) {
  hipLaunchKernelGGL(k_motion_stats, dim3(g.n_cams * 2 * g.n_blocks), dim3(kThreads), 0, st, g, fp, pp, b, rm);
  return hipGetLastError();
}

hipError_t launch_estimate_removal(const Geo& g, const Bufs& b, const Removal& rm, hipStream_t st) {
  const int total = g.n_cams * 2 * g.n_blocks * kCS;
  hipLaunchKernelGGL(k_estimate_removal, dim3((total + kThreads - 1) / kThreads), dim3(kThreads), 0, st, g, b, rm);
  return hipGetLastError();
}

hipError_t launch_estimate(const Geo& g, const Bufs& b, hipStream_t st) {
  const int total = g.n_cams * 2 * g.n_blocks * kCS;
  if (g.fit == RT_FIT_QUANTILE) {
    constexpr int per = kThreads / kWave;
    hipLaunchKernelGGL(k_estimate_quantile, dim3((total + per - 1) / per), dim3(kThreads), 0, st, g, b);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_estimate, dim3((total + kThreads - 1) / kThreads), dim3(kThreads), 0, st, g, b);
  return hipGetLastError();
}

hipError_t launch_weights(const Geo& g, const Bufs& b, hipStream_t st) {
  const int64_t n = (int64_t)g.n_cams * g.w_max;
  hipLaunchKernelGGL(k_weights, dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0, st, g, b);
  return hipGetLastError();
}

hipError_t launch_build_lut(const Geo& g, const Bufs& b, hipStream_t st) {
  hipLaunchKernelGGL(k_build_lut, dim3(g.n_cams * 2 * g.n_blocks), dim3(kThreads), 0, st, g, b);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t n = (int64_t)g.n_cams * g.w_max;
  hipLaunchKernelGGL(k_weights, dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0, st, g, b);
  return hipGetLastError();
}

}  // namespace rc
