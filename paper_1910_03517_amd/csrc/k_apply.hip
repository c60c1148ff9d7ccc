// Apply kernel of section 3.1, weights read from the caller's table.  With
// statistics, each run adds its input histogram and sums to the camera's
// whole-frame statistics with atomics.
#include <hip/hip_ext.h>

#include "dev_apply.h"

namespace rc {

#ifndef RC_APPLY_WAVES
#define RC_APPLY_WAVES 5
#endif
// Workgroup w takes its run of rows (apply_run); no workgroup waits for
// another.  VBLEND: the maps of adjacent blocks blended row by row (a kernel
// of its own, so that its registers do not weigh on the plain pass).
template <bool WRITE, bool STATS, bool VBLEND>
__global__ __launch_bounds__(kApplyThreads) __attribute__((amdgpu_waves_per_eu(RC_APPLY_WAVES)))
void k_apply(Geo g, FramePtrs fp, Bufs b) {
  __shared__ ApplyLds L;
  apply_run<WRITE, STATS, VBLEND, false>(g, fp, b, nullptr, (int)blockIdx.x, L);
}

// Apply with statistics of several frame-sets of the rig (see SetPtrs): the
// same runs as k_apply, once per set, set-major, so that one launch has no
// drain between the frame-sets it holds.
template <bool VBLEND>
__global__ __launch_bounds__(kApplyThreads) __attribute__((amdgpu_waves_per_eu(RC_APPLY_WAVES)))
void k_apply_sets(Geo g, SetPtrs sp) {
  __shared__ ApplyLds L;
  const int f = (int)blockIdx.x / g.n_wg, w = (int)blockIdx.x - f * g.n_wg;
  Bufs b{};
  b.whole_hist = sp.b[f].whole_hist;
  b.whole_sums = sp.b[f].whole_sums;
  b.lut8 = sp.b[f].lut8;
  b.q16 = sp.b[f].q16;
  b.weights = sp.b[f].weights;
  apply_run<true, true, VBLEND, false>(g, sp.f[f], b, nullptr, w, L);
}

// start / stop (may be NULL): events that take the dispatch's own start and
// end times (no marker packets around it).
hipError_t launch_apply(const Geo& g, const FramePtrs& fp, const Bufs& b, bool write, bool stats, hipStream_t st,
                        hipEvent_t start, hipEvent_t stop) {
  const dim3 grid(g.n_wg), block(kApplyThreads);
  if (g.vblend && write && stats)
    hipExtLaunchKernelGGL((k_apply<true, true, true>), grid, block, 0, st, start, stop, 0u, g, fp, b);
  else if (g.vblend && write)
    hipExtLaunchKernelGGL((k_apply<true, false, true>), grid, block, 0, st, start, stop, 0u, g, fp, b);
  else if (write && stats)
    hipExtLaunchKernelGGL((k_apply<true, true, false>), grid, block, 0, st, start, stop, 0u, g, fp, b);
  else if (write)
    hipExtLaunchKernelGGL((k_apply<true, false, false>), grid, block, 0, st, start, stop, 0u, g, fp, b);
  else if (stats)
    hipExtLaunchKernelGGL((k_apply<false, true, false>), grid, block, 0, st, start, stop, 0u, g, fp, b);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

const void* apply_kernel(const Geo& g, bool write, bool stats) {
  if (g.vblend && write && stats) return reinterpret_cast<const void*>(&k_apply<true, true, true>);
  if (g.vblend && write) return reinterpret_cast<const void*>(&k_apply<true, false, true>);
  if (write && stats) return reinterpret_cast<const void*>(&k_apply<true, true, false>);
  if (write) return reinterpret_cast<const void*>(&k_apply<true, false, false>);
  if (stats) return reinterpret_cast<const void*>(&k_apply<false, true, false>);
  return nullptr;
}

hipError_t launch_apply_sets(const Geo& g, const SetPtrs& sp, hipStream_t st, hipEvent_t start, hipEvent_t stop) {
  if (sp.n_sets < 1 || sp.n_sets > kSetsMax || g.n_cams > kSetCams) return hipErrorInvalidValue;
  const dim3 grid(g.n_wg * sp.n_sets), block(kApplyThreads);
  if (g.vblend) hipExtLaunchKernelGGL((k_apply_sets<true>), grid, block, 0, st, start, stop, 0u, g, sp);
  else hipExtLaunchKernelGGL((k_apply_sets<false>), grid, block, 0, st, start, stop, 0u, g, sp);
  return hipGetLastError();
}

}  // namespace rc
