// Cross-channel 3x3 maps (section 5 proposes linear maps across the colour
// channels instead of one affine map per channel): the cross sums of every
// band, the fit of M and t per (camera, side, block), their Q16 form, and the
// apply pass, for rigs of 8-bit RGB cameras.
//
// Fit of one side: mu and the covariance C from the exact sums (binary64),
// the Cholesky factors L_own, L_fac of both bands, the shared factor
// L* = (L_own + L_fac) / 2 and mean mu* = (mu_own + mu_fac) / 2, then
// M = L* L_own^-1 (M L_own = L* solved row by row from the last column) and
// t = mu* - M mu_own.  Every step is one binary64 operation in the written
// order, contraction off.  When either covariance has a pivot <= 0, or M has
// a diagonal entry outside [a_min, a_max] or an off-diagonal entry beyond
// a_max in magnitude, the side takes the per-channel fits of the plain
// estimate instead (a diagonal M).
#include "dev_apply.h"

#pragma clang fp contract(off)

namespace rc {

// ----------------------------------------------------------------- statistics

// Cross sums of the band of unit (k, s, j) = blockIdx.x, one workgroup each.
__global__ __launch_bounds__(kThreads) void k_cross_stats(Geo g, FramePtrs fp, CrossBufs x) {
  __shared__ unsigned long long red[3 * 16];
  const int nb = g.n_blocks, unit = blockIdx.x;
  const int k = unit / (2 * nb), s = (unit / nb) & 1, j = unit % nb;
  if (!cam_active(g, k)) return;
  const DevCam cam = uniform_cam(g, k);
  const int r0 = (int)((int64_t)j * cam.height / nb), r1 = (int)((int64_t)(j + 1) * cam.height / nb);
  const int band = cam.band, c0 = s == 0 ? 0 : cam.width - band;
  const __amdgpu_buffer_rsrc_t rin = frame_rsrc(fp.in[k], cam);
  const int pitch = (int)cam.pitch;
  unsigned long long p01 = 0, p02 = 0, p12 = 0;
  const int total = (r1 - r0) * band;
  for (int i = threadIdx.x; i < total; i += kThreads) {
    const int row = r0 + i / band, col = c0 + i % band;
    const int off = row * pitch + col * 3;
    const uint32_t x0 = __builtin_amdgcn_raw_buffer_load_b8(rin, off, 0, 0);
    const uint32_t x1 = __builtin_amdgcn_raw_buffer_load_b8(rin, off + 1, 0, 0);
    const uint32_t x2 = __builtin_amdgcn_raw_buffer_load_b8(rin, off + 2, 0, 0);
    p01 += x0 * x1;
    p02 += x0 * x2;
    p12 += x1 * x2;
  }
  block_sums(
      3, [&](int i) -> unsigned long long { return i == 0 ? p01 : (i == 1 ? p02 : p12); },
      [&](int i, unsigned long long tot) { x.cross[(int64_t)unit * 3 + i] = tot; }, red);
}

// ----------------------------------------------------------------- estimate

struct MeanCov {
  double mu[3];
  double cov[3][3];
};

// sums: (n, S1, S2) of channels 0..2; cross: (S_RG, S_RB, S_GB).
__device__ inline MeanCov mean_cov(const uint64_t* sums, const uint64_t* cross) {
  MeanCov m;
  const double n = (double)sums[0];
  for (int c = 0; c < 3; ++c) m.mu[c] = (double)sums[c * 3 + 1] / n;
  for (int c = 0; c < 3; ++c) {
    const double ex = (double)sums[c * 3 + 2] / n;
    const double m2 = m.mu[c] * m.mu[c];
    const double v = ex - m2;
    m.cov[c][c] = v > 0.0 ? v : 0.0;
  }
  const int pa[3] = {0, 0, 1}, pb[3] = {1, 2, 2};
  for (int i = 0; i < 3; ++i) {
    const double ex = (double)cross[i] / n;
    const double m2 = m.mu[pa[i]] * m.mu[pb[i]];
    m.cov[pa[i]][pb[i]] = m.cov[pb[i]][pa[i]] = ex - m2;
  }
  return m;
}

// Lower Cholesky factor of C; false when a pivot is not positive.
__device__ inline bool cholesky3(const double (&C)[3][3], double (&L)[3][3]) {
  for (int r = 0; r < 3; ++r)
    for (int c = 0; c < 3; ++c) L[r][c] = 0.0;
  if (!(C[0][0] > 0.0)) return false;
  L[0][0] = __builtin_sqrt(C[0][0]);
  L[1][0] = C[1][0] / L[0][0];
  L[2][0] = C[2][0] / L[0][0];
  const double p11 = C[1][1] - L[1][0] * L[1][0];
  if (!(p11 > 0.0)) return false;
  L[1][1] = __builtin_sqrt(p11);
  L[2][1] = (C[2][1] - L[2][0] * L[1][0]) / L[1][1];
  const double p22 = (C[2][2] - L[2][0] * L[2][0]) - L[2][1] * L[2][1];
  if (!(p22 > 0.0)) return false;
  L[2][2] = __builtin_sqrt(p22);
  return true;
}

// (M, t) of the own side into m[12]; false when a band is empty.
__device__ inline bool fit_cross(const Geo& g, const uint64_t* os, const uint64_t* ox, const uint64_t* fs,
                                 const uint64_t* fx, double (&m)[kX3]) {
  if (os[0] == 0 || fs[0] == 0) return false;
  const MeanCov mo = mean_cov(os, ox), mf = mean_cov(fs, fx);
  double Lo[3][3], Lf[3][3], M[3][3];
  bool ok = cholesky3(mo.cov, Lo);
  ok = cholesky3(mf.cov, Lf) && ok;
  if (ok) {
    for (int r = 0; r < 3; ++r) {
      double ls[3];
      for (int c = 0; c < 3; ++c) ls[c] = (Lo[r][c] + Lf[r][c]) / 2.0;
      const double m2 = ls[2] / Lo[2][2];
      const double m1 = (ls[1] - m2 * Lo[2][1]) / Lo[1][1];
      const double m0 = ((ls[0] - m1 * Lo[1][0]) - m2 * Lo[2][0]) / Lo[0][0];
      M[r][0] = m0;
      M[r][1] = m1;
      M[r][2] = m2;
    }
    for (int r = 0; r < 3; ++r)
      for (int c = 0; c < 3; ++c) {
        const double v = M[r][c];
        const bool good = r == c ? (v >= g.a_min && v <= g.a_max) : (v >= -g.a_max && v <= g.a_max);
        ok = ok && good;
      }
  }
  if (!ok) {
    for (int i = 0; i < kX3; ++i) m[i] = 0.0;
    for (int c = 0; c < 3; ++c) {
      double a, bb;
      (void)fit_sums(g, 3, c, os + c * 3, fs + c * 3, a, bb);
      m[c * 4] = a;
      m[9 + c] = bb;
    }
    return true;
  }
  for (int r = 0; r < 3; ++r) {
    const double mus = (mo.mu[r] + mf.mu[r]) / 2.0;
    const double mx = (M[r][0] * mo.mu[0] + M[r][1] * mo.mu[1]) + M[r][2] * mo.mu[2];
    for (int c = 0; c < 3; ++c) m[r * 3 + c] = M[r][c];
    m[9 + r] = mus - mx;
  }
  return true;
}

// The state p (12 parameters; had: it holds an estimate) of a unit after its
// fit m (fresh) or without one; returns its new valid flag.
__device__ inline uint8_t cross_step(const Geo& g, bool faces, bool fresh, bool had, const double (&m)[kX3],
                                     double (&p)[kX3]) {
  if (!fresh) {
    if (faces && had) return 1;                 // no estimate: keep the state
    for (int i = 0; i < kX3; ++i) p[i] = (i < 9 && i % 4 == 0) ? 1.0 : 0.0;
    return faces ? 0 : 1;                       // identity without a facing band
  }
  const bool blend = g.mode == RT_MODE_SMOOTHING && had;
  const double keep = 1.0 - g.alpha;
  for (int i = 0; i < kX3; ++i) {
    const double tp = keep * p[i];
    const double tn = g.alpha * m[i];
    p[i] = blend ? tp + tn : m[i];
  }
  return 1;
}

// One thread per (camera, side, block): fit, then the temporal step.
__global__ __launch_bounds__(kThreads) void k_estimate_cross(Geo g, Bufs b, CrossBufs x) {
  const int nb = g.n_blocks;
  const int u = blockIdx.x * kThreads + threadIdx.x;
  if (u >= g.n_cams * 2 * nb) return;
  const int k = u / (2 * nb), s = (u / nb) & 1, j = u % nb;
  if (!cam_active(g, k)) return;
  const DevCam& cam = g.cams[k];
  double p[kX3], m[kX3];
  for (int i = 0; i < kX3; ++i) p[i] = x.params3[(int64_t)u * kX3 + i];
  const int fc = cam.face_cam[s];
  const int64_t uf = fc < 0 ? -1 : ((int64_t)fc * 2 + cam.face_side[s]) * nb + j;
  const bool fresh = uf >= 0 && fit_cross(g, b.band_sums + (int64_t)u * kCS * 3, x.cross + (int64_t)u * 3,
                                          b.band_sums + uf * kCS * 3, x.cross + uf * 3, m);
  x.valid3[u] = cross_step(g, uf >= 0, fresh, x.valid3[u] != 0, m, p);
  for (int i = 0; i < kX3; ++i) x.params3[(int64_t)u * kX3 + i] = p[i];
}

// Band statistics, cross sums, fit and fixed-point maps of a frame-set in one
// launch, one workgroup of NT threads per seam block (see Seam; the whole-frame
// statistics that the apply accumulates are cleared here too): the same
// results as k_band_stats, k_cross_stats, k_estimate_cross, k_build_cross and
// k_weights in sequence, which took 35 us of launches and dependent reads
// beside the 62 us apply of the 14x1920x1080 rig; this takes 9 us.
template <int NT>
__global__ __launch_bounds__(NT) void k_seam_cross(Geo g, FramePtrs fp, Bufs b, CrossBufs x) {
  __shared__ BandLds<kBandRep> bands[2];
  __shared__ uint64_t sums[3][9], cross[3][9];
  const int nb = g.n_blocks, tid = threadIdx.x;
  const int k = (int)blockIdx.x / nb, j = (int)blockIdx.x - k * nb;
  zero_whole(g, b, blockIdx.x * NT + tid, gridDim.x * NT);
  if (!cam_active(g, k)) return;
  const DevCam cam = uniform_cam(g, k);
  const Seam sm = seam_of(g, cam, k, j);
  // Thread 64 t fits unit t; its state is read ahead of the band passes.
  const int t = tid / kWave;
  const bool fitter = tid % kWave == 0 && t < sm.n;
  const int u = t == 0 ? sm.u[0] : (t == 1 ? sm.u[1] : sm.u[2]);
  double p[kX3], m[kX3];
  bool had = false;
  if (fitter) {
    for (int i = 0; i < kX3; ++i) p[i] = x.params3[(int64_t)u * kX3 + i];
    had = x.valid3[u] != 0;
  }
  seam_bands<NT, kBandCross>(g, fp, b, BandArgs{nullptr, nullptr, x.cross}, sm, bands, sums, cross);
  if (fitter) {
    const bool faces = sm.faces && t < 2;
    const int o = t == 0 ? 1 : 0;
    const bool fresh = faces && fit_cross(g, sums[t], cross[t], sums[o], cross[o], m);
    x.valid3[u] = cross_step(g, faces, fresh, had, m, p);
    for (int i = 0; i < kX3; ++i) {
      x.params3[(int64_t)u * kX3 + i] = p[i];
      x.q3[(int64_t)u * kX3 + i] = q16_of(p[i]);
    }
  }
  // The camera's blend weights, shared by its seam blocks.
  const int w1 = (int)((int64_t)(j + 1) * g.w_max / nb);
  for (int col = (int)((int64_t)j * g.w_max / nb) + tid; col < w1; col += NT)
    x.weights[(int64_t)k * g.w_max + col] = (uint16_t)blend_weight(cam.width, col);
}

// q3 = round_half_even(params3 * 65536), one thread per parameter.
__global__ __launch_bounds__(kThreads) void k_build_cross(Geo g, CrossBufs x) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= (int64_t)g.n_cams * 2 * g.n_blocks * kX3) return;
  if (!cam_active(g, (int)(i / ((int64_t)2 * g.n_blocks * kX3)))) return;
  x.q3[i] = q16_of(x.params3[i]);
}

// ----------------------------------------------------------------- apply

template <bool STATS>
__global__ __launch_bounds__(kApplyThreads) void k_apply_cross(Geo g, FramePtrs fp, Bufs b, CrossBufs x) {
  __shared__ ApplyLds L;
  b.weights = x.weights;
  apply_run<true, STATS, false, true>(g, fp, b, x.q3, (int)blockIdx.x, L);
}

// ----------------------------------------------------------------- launchers

hipError_t launch_cross_stats(const Geo& g, const FramePtrs& fp, const CrossBufs& x, hipStream_t st) {
  hipLaunchKernelGGL(k_cross_stats, dim3(g.n_cams * 2 * g.n_blocks), dim3(kThreads), 0, st, g, fp, x);
  return hipGetLastError();
}

hipError_t launch_seam_cross(const Geo& g, const FramePtrs& fp, const Bufs& b, const CrossBufs& x, hipStream_t st) {
  constexpr int kNT = 512;
  hipLaunchKernelGGL(k_seam_cross<kNT>, dim3(g.n_cams * g.n_blocks), dim3(kNT), 0, st, g, fp, b, x);
  return hipGetLastError();
}

hipError_t launch_estimate_cross(const Geo& g, const Bufs& b, const CrossBufs& x, hipStream_t st) {
  const int n = g.n_cams * 2 * g.n_blocks;
  hipLaunchKernelGGL(k_estimate_cross, dim3((n + kThreads - 1) / kThreads), dim3(kThreads), 0, st, g, b, x);
  return hipGetLastError();
}

hipError_t launch_build_cross(const Geo& g, const CrossBufs& x, hipStream_t st) {
  const int64_t n = (int64_t)g.n_cams * 2 * g.n_blocks * kX3;
  hipLaunchKernelGGL(k_build_cross, dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0, st, g, x);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  Bufs b{};
  b.weights = x.weights;
  return launch_weights(g, b, st);
}

hipError_t launch_apply_cross(const Geo& g, const FramePtrs& fp, const Bufs& b, const CrossBufs& x, bool stats,
                              hipStream_t st) {
  if (stats) hipLaunchKernelGGL(k_apply_cross<true>, dim3(g.n_wg), dim3(kApplyThreads), 0, st, g, fp, b, x);
  else hipLaunchKernelGGL(k_apply_cross<false>, dim3(g.n_wg), dim3(kApplyThreads), 0, st, g, fp, b, x);
  return hipGetLastError();
}

}  // namespace rc
