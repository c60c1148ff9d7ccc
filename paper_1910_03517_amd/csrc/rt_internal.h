// Internal declarations of the ringcorr HIP library (not part of the C-ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/ringcorr.h"
#include "apply_split.h"

namespace rc {

constexpr int kCS = RT_CSLOTS;   // channel slots
constexpr int kNB = RT_NBINS;    // histogram bins
constexpr int kThreads = 256;    // threads of a workgroup, where a kernel names no other number
constexpr int kMlpIn = RT_MLP_IN, kMlpHid = RT_MLP_HID, kMlpOut = RT_MLP_OUT;

#ifndef RC_APPLY_THREADS
#define RC_APPLY_THREADS 512
#endif
constexpr int kApplyThreads = RC_APPLY_THREADS;   // threads of an apply workgroup

// Per-camera geometry as the kernels see it (uploaded once per context).
struct DevCam {
  int32_t width, height, channels, bit_depth;
  int32_t bps;           // bytes per sample: 1 or 2
  int32_t band;          // band width clamped to floor(W/2)
  int32_t half;          // floor(W/2)
  int32_t row_bytes;     // width * channels * bps
  int32_t face_cam[2];   // camera facing side s, -1 if none (open chain end)
  int32_t face_side[2];
  int32_t ap_cols;       // 4-pixel groups of a row that an apply workgroup takes side by side
  int32_t ap_lanes;      // rows it takes at a time (ap_cols * ap_lanes <= kApplyThreads)
  int64_t pitch;         // bytes between rows
};

// The run of an apply workgroup: rows from row row0 of camera cam0 up to row
// row1 (exclusive) of camera cam1, whole cameras between them.  stride > 0: the
// rows of one camera as RowRun has them; then trow0 and trow1 bound the
// contiguous rows that the form that stages whole tables takes instead.
struct WgRun {
  int32_t cam0, row0, cam1, row1, stride, trow0, trow1;
};

// Frame pointers of one launch, passed by value as a kernel argument.
struct FramePtrs {
  const uint8_t* in[RT_MAX_CAMS];
  uint8_t* out[RT_MAX_CAMS];
};

// Several frame-sets of one rig in one apply launch: set f takes workgroups
// [f * n_wg, (f + 1) * n_wg), its frames at index [f][k] and its own tables,
// weights and whole-frame buffers (the pipeline's slots).
// Sized so that the kernel argument stays near the single-set one.
constexpr int kSetsMax = 4;    // frame-sets per launch
constexpr int kSetCams = 16;   // cameras per frame-set
struct SetFrames {
  const uint8_t* in[kSetCams];
  uint8_t* out[kSetCams];
};
struct SetBufs {
  uint32_t* whole_hist;
  uint64_t* whole_sums;
  uint8_t* lut8;
  int64_t* q16;
  uint16_t* weights;
};
struct SetPtrs {
  SetFrames f[kSetsMax];
  SetBufs b[kSetsMax];
  int32_t n_sets;
};

// Caller buffers (device pointers) of one launch.
struct Bufs {
  uint32_t* band_hist;
  uint64_t* band_sums;
  uint32_t* whole_hist;
  uint64_t* whole_sums;
  double* params;
  uint8_t* valid;
  uint8_t* lut8;
  int64_t* q16;
  uint16_t* weights;
};

// Caller buffers of the cross-channel 3x3 maps (device pointers).
struct CrossBufs {
  uint64_t* cross;    // [K][2][NB][3] = (S_RG, S_RB, S_GB)
  double* params3;    // [K][2][NB][12] = M row-major, then t
  uint8_t* valid3;    // [K][2][NB]
  int64_t* q3;        // [K][2][NB][12]
  uint16_t* weights;  // [K][w_max]
};

// Context-wide constants passed to every kernel.
struct Geo {
  const DevCam* cams;    // device array [K]
  const WgRun* runs;     // device array [n_wg]; NULL: the default split over a part of the rig
  int32_t n_cams, n_blocks, w_max, n_tiles;
  int32_t mode;
  int32_t n_wg;          // apply workgroups
  double alpha, a_min, a_max;
  uint64_t active;       // cameras processed by this launch (bit k = camera k)
  int32_t vblend;        // 1: the maps of adjacent blocks are blended row by row in the apply
  int32_t fit;           // RT_FIT_MOMENTS or RT_FIT_QUANTILE
};

__host__ __device__ inline bool cam_active(const Geo& g, int k) { return (g.active >> k) & 1ull; }

// Buffer resource over one frame: loads beyond the last sample of the frame
// return zero and stores there are dropped by the hardware range check.
constexpr int kRsrcWord3 = 0x00020000;   // raw dword access on gfx9-family parts

// Values the caller knows to be the same in every lane of the wave, moved to
// scalar registers.  Table entries read from global memory land in vector
// registers; without this a buffer resource built from them would be
// non-uniform and every access through it would be wrapped in a loop over
// the distinct values.
__device__ inline int32_t uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline int64_t uniform(int64_t v) {
  const uint64_t u = (uint64_t)v;
  return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(u >> 32)) << 32) |
                   (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)u));
}
template <typename T>
__device__ inline T* uniform_ptr(T* p) {
  return reinterpret_cast<T*>(uniform((int64_t)reinterpret_cast<uintptr_t>(p)));
}

// A copy of *p, p the same in every lane of the wave, through scalar loads:
// context tables do not change while a kernel runs.
template <typename T>
__device__ inline T uniform_load(const T* p) {
  static_assert(sizeof(T) % 4 == 0, "whole dwords");
  const __attribute__((address_space(4))) int32_t* q =
      (const __attribute__((address_space(4))) int32_t*)(uintptr_t)uniform((int64_t)(uintptr_t)p);
  int32_t v[sizeof(T) / 4];
#pragma unroll
  for (int i = 0; i < (int)(sizeof(T) / 4); ++i) v[i] = q[i];
  T t;
  __builtin_memcpy(&t, v, sizeof t);
  return t;
}
__device__ inline DevCam uniform_cam(const Geo& g, int k) { return uniform_load(g.cams + k); }
__device__ inline WgRun uniform_run(const Geo& g, int w) { return uniform_load(g.runs + w); }

// p and cam must be uniform over the wave (see uniform_cam).
__device__ inline __amdgpu_buffer_rsrc_t frame_rsrc(const void* p, const DevCam& cam) {
  const int64_t bytes = (int64_t)(cam.height - 1) * cam.pitch + cam.row_bytes;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(uniform_ptr(p)), (short)0, uniform((int32_t)bytes),
                                           kRsrcWord3);
}

// Index of a (camera, side, block, channel) unit in the caller layouts.
__host__ __device__ inline int64_t unit_index(int k, int s, int j, int c, int nb) {
  return (((int64_t)k * 2 + s) * nb + j) * kCS + c;
}

// Launchers (each defined next to its kernels).  All return hipError_t of the launch.
hipError_t launch_band_stats(const Geo& g, const FramePtrs& fp, const Bufs& b, hipStream_t st);
hipError_t launch_estimate(const Geo& g, const Bufs& b, hipStream_t st);
// (beside: other kernels run at the same time, as in a pipeline.)
hipError_t launch_band_estimate(const Geo& g, const FramePtrs& fp, const Bufs& b, hipStream_t st, bool beside = false);
hipError_t launch_build_lut(const Geo& g, const Bufs& b, hipStream_t st);
hipError_t launch_apply(const Geo& g, const FramePtrs& fp, const Bufs& b, bool write, bool stats, hipStream_t st,
                        hipEvent_t start = nullptr, hipEvent_t stop = nullptr);
// Host addresses of the kernels that launch_band_estimate and launch_apply
// launch for g (the latter with write and stats as given); both take
// (Geo, FramePtrs, Bufs).  Used to find them among a captured graph's nodes.
const void* band_estimate_kernel(const Geo& g);
const void* apply_kernel(const Geo& g, bool write, bool stats);

// Apply with whole-frame statistics of sp.n_sets (1..kSetsMax) frame-sets of
// the rig in one launch (every camera at most kSetCams; g.active the same
// for all sets).
hipError_t launch_apply_sets(const Geo& g, const SetPtrs& sp, hipStream_t st, hipEvent_t start = nullptr,
                             hipEvent_t stop = nullptr);
hipError_t launch_zero_whole(const Geo& g, const Bufs& b, hipStream_t st);
hipError_t launch_weights(const Geo& g, const Bufs& b, hipStream_t st);
hipError_t launch_cross_stats(const Geo& g, const FramePtrs& fp, const CrossBufs& x, hipStream_t st);
hipError_t launch_seam_cross(const Geo& g, const FramePtrs& fp, const Bufs& b, const CrossBufs& x, hipStream_t st);
hipError_t launch_estimate_cross(const Geo& g, const Bufs& b, const CrossBufs& x, hipStream_t st);
hipError_t launch_build_cross(const Geo& g, const CrossBufs& x, hipStream_t st);
hipError_t launch_apply_cross(const Geo& g, const FramePtrs& fp, const Bufs& b, const CrossBufs& x, bool stats,
                              hipStream_t st);
struct PrevPtrs;
struct Removal;
hipError_t launch_band_estimate_removal(const Geo& g, const FramePtrs& fp, const PrevPtrs& pp, const Bufs& b,
                                        const Removal& rm, hipStream_t st, bool beside = false);
hipError_t launch_motion_stats(const Geo& g, const FramePtrs& fp, const PrevPtrs& pp, const Bufs& b,
                               const Removal& rm, hipStream_t st);
hipError_t launch_estimate_removal(const Geo& g, const Bufs& b, const Removal& rm, hipStream_t st);
hipError_t launch_stream_copy(void* dst, const void* src, int64_t bytes, int vec_bytes, hipStream_t st);
hipError_t launch_attention(const Geo& g, const FramePtrs& fp, const uint8_t* const* prev, uint32_t* cells,
                            uint32_t* windows, uint8_t* selected, int hc, int wc, int cell, int m, uint32_t tau,
                            uint32_t theta, hipStream_t st);
hipError_t launch_seam_cost(const Geo& g, const FramePtrs& fp, double* seam, double* interior, double* rows,
                            int row_stride, int factor, int max_rows, hipStream_t st);

}  // namespace rc
