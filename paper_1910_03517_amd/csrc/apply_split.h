// How the apply pass's default split lays a camera's rows over its workgroups:
// plain integer arithmetic that the kernels and the host share.
#pragma once

#include <stdint.h>

namespace rc {

// The rows of one run of a camera of `height` rows: steps of `lanes` rows
// starting at row0, row0 + stride, ..., those below row1; row1 is the end of
// the run's last row.
struct RowRun {
  int32_t row0, row1, stride;
};

// Whether the m runs of a camera of `steps` steps interleave (run i takes steps
// i, i + m, ...) or lie one after the other (each a contiguous share).
// Interleaved, all of a camera's workgroups read and write side by side in its
// frame, a handful of streams for the memory; but a run then spans all blocks
// and looks at and stages all of their maps, so it needs as many steps as there
// are blocks.  Apply with statistics on MI355X, us interleaved and contiguous:
// 14x1920x1080, 30 steps a run, 16 blocks 43.2 and 44.0; 4x4096x2160, 34 steps,
// 50.2 and 52.1; one 1920x1080 image, 3 steps, 16.3 and 14.4; 14x1920x1080 of 256
// blocks 59.7 and 45.0, of 64 blocks 44.7 and 44.4.
__host__ __device__ inline bool runs_interleave(int steps, int m, int n_blocks) { return steps / m >= n_blocks; }

// Run i of the m runs (m <= steps) of a camera, in steps of `lanes` rows.
__host__ __device__ inline RowRun row_run(int height, int lanes, int i, int m, bool interleave) {
  const uint32_t steps = (uint32_t)(height + lanes - 1) / (uint32_t)lanes;
  RowRun r;
  uint32_t end;                                   // the step after the run's last
  if (interleave) {
    r.row0 = i * lanes;
    r.stride = m * lanes;
    end = (uint32_t)i + (steps - 1 - (uint32_t)i) / (uint32_t)m * (uint32_t)m + 1;
  } else {                                        // (steps * m below 2^31: at most 32768 and 65536)
    r.row0 = (int)((uint32_t)i * steps / (uint32_t)m) * lanes;
    r.stride = lanes;
    end = ((uint32_t)i + 1) * steps / (uint32_t)m;
  }
  r.row1 = (int)end * lanes < height ? (int)end * lanes : height;
  return r;
}

// The workgroups of the default split shared among the cameras of the bit mask
// `active`, by their bytes, at least one each and at most one a step: camera
// k's runs are workgroups first[k] .. first[k + 1] - 1 (`first` holds n + 1
// entries).  Returns their number, at most max(total, active cameras).
inline int split_shares(int n, const int64_t* bytes, const int32_t* steps, uint64_t active, int total,
                        uint16_t* first) {
  int64_t all = 0, before = 0;
  int cams = 0;
  for (int k = 0; k < n; ++k)
    if ((active >> k) & 1u) all += bytes[k], ++cams;
  const int64_t more = total > cams ? total - cams : 0;      // beyond one each
  int w = 0;
  for (int k = 0; k < n; ++k) {
    first[k] = (uint16_t)w;
    if (!((active >> k) & 1u)) continue;
    const int64_t a = more * before / all, e = more * (before + bytes[k]) / all;
    before += bytes[k];
    const int m = 1 + (int)(e - a);
    w += m < steps[k] ? m : steps[k];
  }
  first[n] = (uint16_t)w;
  return w;
}

}  // namespace rc
