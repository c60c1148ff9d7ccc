// Difference approach of section 3.3's attention mechanisms: the absolute
// difference of two consecutive frames, thresholded (a pixel is on when the
// difference exceeds tau << (bit_depth - 8) on some channel), counted per
// cell of c x c pixels, then summed over every window of m x m cells; a
// window is selected when its count exceeds theta.  Exact integers.
//
// k_diff_cells: one workgroup per (camera, cell row), its threads laid over the
// rows as the apply pass lays them: a thread takes groups of 4 consecutive
// pixels (c is a multiple of 4, so a group lies in one cell), kAttnRows rows of
// both frames in flight, counts its on-pixels and adds the count to its cell in
// LDS; the cell row is then written out.  Both frames are read once: 2 x
// (samples x bytes) per pixel, which is what bounds it.
// k_windows: one workgroup per (camera, kWinRows rows of windows, chunk of
// columns): a thread sums its column's cells over each window's rows, then m
// neighbouring column sums from LDS make a window; it is bound by latency.
// Measured on MI355X, 14x1920x1080 RGB8, cells of 16, m = 8: one row of a
// group at a time and m x m cells per window 43.6 us in all, this 36.1 us (4.8
// TB/s).
// Outputs are laid out over the largest camera's grid; entries beyond a
// camera's own cells or windows are written as zero (not selected).
#include "dev_apply.h"

namespace rc {

struct AttnArgs {
  const uint8_t* prev[RT_MAX_CAMS];
  uint32_t* cells;      // [K][hc][wc]
  uint32_t* windows;    // [K][hc - m + 1][wc - m + 1] or null
  uint8_t* selected;    // same shape or null
  int32_t hc, wc;       // padded cell grid of every camera
  int32_t cell, m;
  uint32_t tau, theta;  // tau in 8-bit units
};

constexpr int kAttnMaxCells = 32768 / 4;   // cells of one cell row for the widest frame and c = 4

struct AttnLds {
  uint32_t cnt[kAttnMaxCells];
};

constexpr int kAttnRows = 4;   // rows of both frames in flight per thread

// On-pixels among the first npx pixels of a group of the two frames.
template <int C, int BPS>
__device__ inline uint32_t group_on(const uint32_t (&a)[C * BPS], const uint32_t (&b)[C * BPS], int npx,
                                    uint32_t thr) {
  uint32_t on = 0;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    uint32_t d = 0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const uint32_t x = group_sample<BPS>(a, p * C + c), y = group_sample<BPS>(b, p * C + c);
      const uint32_t e = x > y ? x - y : y - x;
      d = d > e ? d : e;
    }
    on += p < npx && d > thr ? 1u : 0u;
  }
  return on;
}

template <int C, int BPS>
__device__ void diff_cell_row(const DevCam& cam, const FramePtrs& fp, const AttnArgs& a, int k, int ci,
                              AttnLds& L) {
  constexpr int NW = C * BPS;
  const int tid = threadIdx.x;
  const int W = cam.width, H = cam.height, c = a.cell;
  const int ncell = (W + c - 1) / c;
  for (int i = tid; i < ncell; i += kApplyThreads) L.cnt[i] = 0;
  __syncthreads();
  const __amdgpu_buffer_rsrc_t ra = frame_rsrc(fp.in[k], cam);
  const __amdgpu_buffer_rsrc_t rb = frame_rsrc(a.prev[k], cam);
  const uint32_t thr = a.tau << (cam.bit_depth - 8);
  const int pitch = (int)cam.pitch;
  const int r0 = ci * c, r1 = min(H, r0 + c);
  const int ngroups = (W + 3) >> 2;
  const int cols = cam.ap_cols, step = cam.ap_lanes;
  const int ln = tid / cols;
  for (int g = tid - ln * cols; ln < step && g < ngroups; g += cols) {
    const int col0 = g * 4, npx = min(4, W - col0);
    uint32_t n = 0;
    for (int r = r0 + ln; r < r1; r += kAttnRows * step) {
      uint32_t x[kAttnRows][NW], y[kAttnRows][NW];
#pragma unroll
      for (int u = 0; u < kAttnRows; ++u) {
        if (r + u * step < r1) {
          const int off = (r + u * step) * pitch + col0 * NW;
          if (npx == 4) {
            load_group<NW>(ra, off, x[u]);
            load_group<NW>(rb, off, y[u]);
          } else {
            load_part<NW>(ra, off, npx * NW, x[u]);
            load_part<NW>(rb, off, npx * NW, y[u]);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < kAttnRows; ++u)
        if (r + u * step < r1) n += group_on<C, BPS>(x[u], y[u], npx, thr);
    }
    if (n) atomicAdd(&L.cnt[col0 / c], n);
  }
  __syncthreads();
  uint32_t* out = a.cells + ((int64_t)k * a.hc + ci) * a.wc;
  for (int i = tid; i < a.wc; i += kApplyThreads) out[i] = i < ncell ? L.cnt[i] : 0u;
}

__global__ __launch_bounds__(kApplyThreads) void k_diff_cells(Geo g, FramePtrs fp, AttnArgs a) {
  __shared__ AttnLds L;
  const int k = blockIdx.y, ci = blockIdx.x;
  if (!cam_active(g, k)) return;
  const DevCam cam = uniform_cam(g, k);
  if (ci * a.cell >= cam.height) {   // below the camera's cell grid: zeros
    uint32_t* out = a.cells + ((int64_t)k * a.hc + ci) * a.wc;
    for (int i = threadIdx.x; i < a.wc; i += kApplyThreads) out[i] = 0u;
    return;
  }
  if (cam.bps == 2) diff_cell_row<1, 2>(cam, fp, a, k, ci, L);
  else if (cam.channels == 3) diff_cell_row<3, 1>(cam, fp, a, k, ci, L);
  else diff_cell_row<1, 1>(cam, fp, a, k, ci, L);
}

// Windows of kWinRows rows and kThreads - m + 1 columns.
constexpr int kWinRows = 4;

__global__ __launch_bounds__(kThreads) void k_windows(Geo g, AttnArgs a) {
  __shared__ uint32_t col[kWinRows][kThreads];
  const int k = blockIdx.z;
  if (!cam_active(g, k)) return;
  const int m = a.m, hw = a.hc - m + 1, ww = a.wc - m + 1;
  const int per = kThreads - m + 1;
  const int wy0 = blockIdx.y * kWinRows, wx0 = blockIdx.x * per, tid = threadIdx.x;
  const DevCam cam = uniform_cam(g, k);
  // Windows of this camera's own cell grid; the rest of the padded grid is 0.
  const int hck = (cam.height + a.cell - 1) / a.cell, wck = (cam.width + a.cell - 1) / a.cell;
  const uint32_t* cells = a.cells + (int64_t)k * a.hc * a.wc;
  const int x = wx0 + tid;
  uint32_t s[kWinRows];
#pragma unroll
  for (int r = 0; r < kWinRows; ++r) s[r] = 0;
  if (x < wck) {
    // Cell row wy0 + y belongs to the windows of rows max(0, y - m + 1) .. y.
    for (int y = 0; y < m + kWinRows - 1 && wy0 + y < hck; ++y) {
      const uint32_t v = cells[(wy0 + y) * a.wc + x];
#pragma unroll
      for (int r = 0; r < kWinRows; ++r) s[r] += y >= r && y < r + m ? v : 0u;
    }
  }
#pragma unroll
  for (int r = 0; r < kWinRows; ++r) col[r][tid] = s[r];
  __syncthreads();
  const int wx = wx0 + tid;
  if (tid >= per || wx >= ww) return;
#pragma unroll
  for (int r = 0; r < kWinRows; ++r) s[r] = 0;
  for (int d = 0; d < m; ++d) {
#pragma unroll
    for (int r = 0; r < kWinRows; ++r) s[r] += col[r][tid + d];
  }
#pragma unroll
  for (int r = 0; r < kWinRows; ++r) {
    const int wy = wy0 + r;
    if (wy >= hw) continue;
    const bool inside = wy + m <= hck && wx + m <= wck;
    const uint32_t n = inside ? s[r] : 0u;
    const int64_t o = (int64_t)k * hw * ww + (int64_t)wy * ww + wx;
    if (a.windows) a.windows[o] = n;
    if (a.selected) a.selected[o] = inside && n > a.theta ? 1 : 0;
  }
}

hipError_t launch_attention(const Geo& g, const FramePtrs& fp, const uint8_t* const* prev, uint32_t* cells,
                            uint32_t* windows, uint8_t* selected, int hc, int wc, int cell, int m, uint32_t tau,
                            uint32_t theta, hipStream_t st) {
  AttnArgs a{};
  for (int k = 0; k < g.n_cams; ++k) a.prev[k] = prev[k];
  a.cells = cells;
  a.windows = windows;
  a.selected = selected;
  a.hc = hc;
  a.wc = wc;
  a.cell = cell;
  a.m = m;
  a.tau = tau;
  a.theta = theta;
  hipLaunchKernelGGL(k_diff_cells, dim3(hc, g.n_cams), dim3(kApplyThreads), 0, st, g, fp, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int hw = hc - m + 1, ww = wc - m + 1, per = kThreads - m + 1;
  if (hw > 0 && ww > 0 && (windows || selected)) {
    const dim3 grid((ww + per - 1) / per, (hw + kWinRows - 1) / kWinRows, g.n_cams);
    hipLaunchKernelGGL(k_windows, grid, dim3(kThreads), 0, st, g, a);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace rc
