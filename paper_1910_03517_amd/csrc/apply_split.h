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

constexpr int kSplitBlocks = 64;   // blocks whose maps a workgroup stages at a time (8-bit affine ones)

// Whether the m runs of a camera of `steps` steps interleave (run i takes steps
// i, i + m, ...) or lie one after the other (each a contiguous share).
// Interleaved, all of a camera's workgroups read and write side by side in its
// frame, a handful of streams for the memory; but a run then spans all blocks
// and stages all of their maps.  That is worth it from four steps a run on if
// the maps are staged at once, and else from as many steps as blocks.  Apply with
// statistics on MI355X, us interleaved and contiguous: 14x1920x1080, 30 steps a
// run, 16 blocks 43.2 and 44.0; 4x4096x2160, 34 steps, 50.2 and 52.1; sixteen
// 1280x720, 7 steps, 27.3 and 30.2; one 1280x720, 3 steps, 10.9 and 10.0;
// 14x1920x1080 of 256 blocks 59.7 and 45.0.
__host__ __device__ inline bool runs_interleave(int steps, int m, int n_blocks) {
  const int run = steps / m;
  return run >= n_blocks || (run >= 4 && n_blocks <= kSplitBlocks);
}

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

constexpr int kSplitMany = 512, kSplitFew = 256;   // apply workgroups: two per compute unit, one
constexpr int kSplitRows = 6;                      // steps a thread has in flight

// The forms in which a thread evaluates a row's maps (see dev_apply.h), and the
// rows of each it has in flight.  Whether a form is rare decides, not what it
// costs in registers alone: every 16-bit camera takes kMapWide with one channel,
// every 8-bit rt_apply without statistics kMapTable (55 registers with two
// rows, 67 with six).  Two rows and six, us: eight 1920x1080 cameras of 16 bits
// with statistics 23.6 and 22.3, without 17.8 and 16.5, blended maps 22.1 and
// 20.2; eight of 8-bit gray without statistics 14.0 and 11.4.  The exact forms of
// 8-bit maps keep two: their 64-bit maps of three channels would not fit the
// registers beside six rows.
enum { kMapDirect, kMapWide, kMapTable, kMapCross, kMapCrossWide };
constexpr int rows_in_flight(int kind, int channels, bool stats) {
  return kind == kMapDirect || kind == kMapCross || (kind == kMapWide && channels == 1) || (kind == kMapTable && !stats)
             ? kSplitRows : 2;
}

// Apply workgroups of the default split for `steps` steps over all cameras.  A
// workgroup beyond one per compute unit pays its set-up and the atomics of its
// histogram's flush, all of a camera's on the same 768 words, and is worth it
// only for work that one per compute unit has not in flight after two rounds.
// MI355X, apply with statistics, us with 256 and 512 workgroups: one 1920x1080
// image (1080 steps) 11.9 and 14.4, three 640x480 (480) 10.2 and 13.4, two
// 1920x1080 (2160) 16.2 and 17.3, five 1031x517 (2585) 16.3 and 16.4, six
// 1280x720 (4320) 17.7 and 17.9, eight 1920x1080 of 16 bits (8640) 27.1 and 22.8,
// fourteen 1920x1080 (15120) 47.3 and 42.9 (768 workgroups: 51.7).
__host__ __device__ inline int split_total(int64_t steps) { return steps <= 2 * kSplitRows * kSplitFew ? kSplitFew : kSplitMany; }

// How a workgroup of `threads` threads lies over the rows of a camera of `height`
// rows of `groups` groups of 4 pixels, when `share` workgroups take the camera:
// `cols` groups of `lanes` rows (at most max_lanes), a row in equal column
// chunks.  A thread walks the chunks one after the other and in each its run's
// steps, kSplitRows of them in flight.  The split of the least cost: the steps
// of all chunks, two for each serial trip to memory, and two for a chunk (its
// weights, and rows in pieces for the memory); of equal ones the fewest chunks.
// Apply with statistics, us, laid by busy threads / by trips alone / so:
// 640x480 32 x 16 in five chunks (512 threads busy, 30 workgroups) 12.4 and
// otherwise 160 x 3 in one (480 threads, 160 workgroups) 8.8; six 1280x720 of 64
// blocks 22.8 / 17.9 / 16.8 (without statistics 19.7 / 10.5 / 13.4: the table form
// stages its tables once a chunk), sixteen of 16 blocks 29.2 / 32.5 / 27.4 (64 x 8, 107 x
// 4, 160 x 3), thirty-two 46.3 / 52.0 / 43.8; twenty 1600x900 53.2 / 55.6 / 45.7
// (100 x 5, 80 x 6, 400 x 1); sixteen 1031x517 26.5 / 23.0 / 23.4; fourteen
// 800x600 19.2 / 18.0 / 18.3; and the sum of steps and trips alone 52.3 on six
// 2592x1944 (162 x 4), so 49.5 (216 x 2).
inline void lay_rows(int groups, int height, int share, int max_lanes, int threads, int32_t* cols, int32_t* lanes) {
  int64_t best = -1;
  for (int chunks = 1; chunks <= 8 || best < 0; ++chunks) {
    const int c = (groups + chunks - 1) / chunks;
    if (c > threads) continue;
    const int l = threads / c < max_lanes ? threads / c : max_lanes;
    const int steps = (height + l - 1) / l, m = share < steps ? share : steps;
    const int run = (steps + m - 1) / m;                // steps of a run
    const int64_t cost = (int64_t)chunks * (run + 2 * ((run + kSplitRows - 1) / kSplitRows) + 2);
    if (best < 0 || cost < best) {
      best = cost;
      *cols = c;
      *lanes = l;
    }
  }
}

// The workgroups of a camera of `bytes` bytes and `steps` steps, the `before` first
// of the `all` bytes of a launch being those of the active cameras ahead of it:
// one, its part by bytes of the `more` beyond one each, and at most one a step.
// In binary64, whose division the kernels do faster than 64-bit integers': the
// products stay below 2^47 and the quotients below 512, so each quotient's floor
// is that of the exact one.
__host__ __device__ inline int camera_share(int more, int64_t before, int64_t bytes, int64_t all, int steps) {
  const double to = (double)more * (double)(before + bytes) / (double)all;
  const double from = (double)more * (double)before / (double)all;
  const int m = 1 + (int)to - (int)from;
  return m < steps ? m : steps;
}

// The default split's workgroups over the cameras of the bit mask `active`:
// camera k's runs are workgroups first[k] .. first[k + 1] - 1 (`first` holds n + 1
// entries).  Returns their number.
inline int split_shares(int n, const int64_t* bytes, const int32_t* steps, uint64_t active, uint16_t* first) {
  int64_t all = 0, all_steps = 0, before = 0;
  int cams = 0, w = 0;
  for (int k = 0; k < n; ++k)
    if ((active >> k) & 1u) all += bytes[k], all_steps += steps[k], ++cams;
  const int more = split_total(all_steps) - cams;
  for (int k = 0; k < n; ++k) {
    first[k] = (uint16_t)w;
    if (!((active >> k) & 1u)) continue;
    w += camera_share(more, before, bytes[k], all, steps[k]);
    before += bytes[k];
  }
  first[n] = (uint16_t)w;
  return w;
}

}  // namespace rc
