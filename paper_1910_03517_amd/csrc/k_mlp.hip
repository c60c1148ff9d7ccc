// Kernels of the learned surrogate's MLP (576 -> 256 -> 256 -> 6, ReLU):
// an FP32 GEMM on the matrix cores with fused bias / ReLU / ReLU-mask
// epilogues and an optional ones row for bias gradients, the MSE gradient and
// value, Adam over the whole network in one launch, and a row gather for
// mini-batches.
#include "dev_mlp.h"

namespace rc {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kGemmTile = 64;   // workgroup tile (rows and columns)
constexpr int kGemmK = 32;      // k-slab staged in LDS
constexpr int kWsMaxRows = 2048;  // up to this many rows, row-major products use the k-split tile kernel

enum { kEpiNone = 0, kEpiBias = 1, kEpiBiasRelu = 2, kEpiMask = 3 };

// C[M][N] (row stride ldc) = A x B with A(i, k) = A[i * sai + k * sak] and
// B(k, j) = B[k * sbk + j * sbj] (strides express transposes), then the
// epilogue: + bias[j]; + bias[j] and ReLU; or times (mask[i][j] > 0).  With
// ones_row non-NULL the product also gets a row M of A equal to all ones, so
// that row M of the result, the column sums of B, is stored to ones_row[j]
// (the bias gradient next to a weight gradient).
// Four waves each own a 32x32 sub-tile and accumulate it with
// v_mfma_f32_32x32x2_f32: lane l supplies A(i = l % 32, k = l / 32) and
// B(k = l / 32, j = l % 32) and holds D(i, j) for j = l % 32 and
// i = 8 (r / 4) + 4 (l / 32) + r % 4 in accumulator register r.  The next
// K-slab is fetched into registers while the current one is multiplied.
template <int EPI>
__device__ __forceinline__ void k_gemm_body(int M, int N, int K, const float* __restrict__ A, int64_t sai,
                                            int64_t sak, const float* __restrict__ B, int64_t sbk, int64_t sbj,
                                            float* __restrict__ C, int ldc, const float* __restrict__ bias,
                                            const float* __restrict__ mask, int ldm, float* __restrict__ ones_row) {
  constexpr int kPer = kGemmK * kGemmTile / 256;   // staged elements per thread and operand
  __shared__ float As[kGemmK][kGemmTile + 1];
  __shared__ float Bs[kGemmK][kGemmTile + 1];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int i0 = blockIdx.y * kGemmTile;
  const int j0 = blockIdx.x * kGemmTile;
  const int wi = (wave >> 1) * 32;
  const int wj = (wave & 1) * 32;
  const int MA = ones_row ? M + 1 : M;             // rows of A including the ones row
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;

  float ra[kPer], rb[kPer];
  // Element e of a staged slab is (kk, ii) with kk fastest when the operand
  // is contiguous along k, ii fastest otherwise, so that consecutive threads
  // read consecutive addresses either way (coalesced loads).
  const bool a_kfast = sak == 1, b_kfast = sbk == 1 && sbj != 1;
  auto slab_pos = [](int e, bool kfast, int& kk, int& ii) {
    if (kfast) { kk = e % kGemmK; ii = e / kGemmK; }
    else { kk = e / kGemmTile; ii = e % kGemmTile; }
  };
  auto fetch = [&](int k0) {
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int e = tid + q * 256;
      int kk, ii;
      slab_pos(e, a_kfast, kk, ii);
      const int gi = i0 + ii, gka = k0 + kk;
      float a = 0.0f;
      if (gka < K) {
        if (gi < M) a = A[(int64_t)gi * sai + (int64_t)gka * sak];
        else if (gi < MA) a = 1.0f;
      }
      ra[q] = a;
      slab_pos(e, b_kfast, kk, ii);
      const int gj = j0 + ii, gkb = k0 + kk;
      rb[q] = (gkb < K && gj < N) ? B[(int64_t)gkb * sbk + (int64_t)gj * sbj] : 0.0f;
    }
  };
  fetch(0);
  for (int k0 = 0; k0 < K; k0 += kGemmK) {
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int e = tid + q * 256;
      int kk, ii;
      slab_pos(e, a_kfast, kk, ii);
      As[kk][ii] = ra[q];
      slab_pos(e, b_kfast, kk, ii);
      Bs[kk][ii] = rb[q];
    }
    __syncthreads();
    if (k0 + kGemmK < K) fetch(k0 + kGemmK);
#pragma unroll
    for (int kk = 0; kk < kGemmK; kk += 2) {
      const float a = As[kk + (lane >> 5)][wi + (lane & 31)];
      const float b = Bs[kk + (lane >> 5)][wj + (lane & 31)];
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0);
    }
    __syncthreads();
  }

  const int j = j0 + wj + (lane & 31);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int i = i0 + wi + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
    if (j >= N) continue;
    if (i < M) {
      float v = acc[r];
      if (EPI == kEpiBias || EPI == kEpiBiasRelu) v += bias[j];
      if (EPI == kEpiBiasRelu) v = v > 0.0f ? v : 0.0f;
      if (EPI == kEpiMask) v = mask[(int64_t)i * ldm + j] > 0.0f ? v : 0.0f;
      C[(int64_t)i * ldc + j] = v;
    } else if (i == M && ones_row) {
      ones_row[j] = acc[r];
    }
  }
}

template <int EPI>
__global__ __launch_bounds__(256) void k_gemm(int M, int N, int K, const float* __restrict__ A, int64_t sai,
                                              int64_t sak, const float* __restrict__ B, int64_t sbk, int64_t sbj,
                                              float* __restrict__ C, int ldc, const float* __restrict__ bias,
                                              const float* __restrict__ mask, int ldm,
                                              float* __restrict__ ones_row) {
  k_gemm_body<EPI>(M, N, K, A, sai, sak, B, sbk, sbj, C, ldc, bias, mask, ldm, ones_row);
}

// The same product for few output rows (every product of the network at
// inference and mini-batch sizes), where 64 x 64 tiles would leave most
// compute units idle and each wave a long serial chain of MFMAs.  A
// workgroup of W waves owns a 32 x 32 tile; wave w sums k over its own range
// [w kw, (w + 1) kw) (kw a multiple of 8) straight from global memory: per 8
// k, lane l supplies A(i, k0 + 4 g + c) and B(k0 + 4 g + c, j) for c = 0..3
// (g = l / 32, i and j = l % 32), the c-th of 4 MFMAs pairing k0 + c with
// k0 + 4 + c.  The loads of kWsChunk such steps are in flight together, and
// the next chunk's are issued before the current chunk's MFMAs.  The waves'
// tiles are added in LDS in wave order, then the epilogue; row M is the ones
// row when ones_row is given (stored without epilogue).  With idx (a training
// step's first layer), row i of A is row idx[i] of the table A.
constexpr int kWsTile = 32;
constexpr int kWsChunk = 4;
template <int EPI, int W>
__global__ __launch_bounds__(W * 64) void k_gemm_wsplit(int M, int N, int K, int kw, const float* __restrict__ A,
                                                        int64_t sai, int64_t sak, const float* __restrict__ B,
                                                        int64_t sbk, int64_t sbj, float* __restrict__ C, int ldc,
                                                        const float* __restrict__ bias, const float* __restrict__ mask,
                                                        int ldm, float* __restrict__ ones_row,
                                                        const int32_t* __restrict__ idx) {
  __shared__ float red[W][16][64];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int g = lane >> 5;
  const int i0 = blockIdx.y * kWsTile, j0 = blockIdx.x * kWsTile;
  const int ia = i0 + (lane & 31), jb = j0 + (lane & 31);
  const bool arow = ia < M, bcol = jb < N;
  const float aone = (ones_row && ia == M) ? 1.0f : 0.0f;   // the ones row, or padding
  const float* pa = A + (int64_t)(arow ? (idx ? idx[ia] : ia) : 0) * sai;
  const float* pb = B + (int64_t)(bcol ? jb : 0) * sbj;
  const int kbeg = wave * kw;
  const int kend = (K - kbeg) < kw ? K : kbeg + kw;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
  float a[kWsChunk][4], b[kWsChunk][4], an[kWsChunk][4], bn[kWsChunk][4];
  // An operand contiguous along k is read 16 bytes per lane (one load for
  // the four k of a step) where the whole quad is in range.
  const bool a_vec = sak == 1, b_vec = sbk == 1;
  auto load = [&](int k0, float (*av)[4], float (*bv)[4]) {
#pragma unroll
    for (int s = 0; s < kWsChunk; ++s) {
      const int kq = k0 + 8 * s + 4 * g;
      const bool quad = kq + 3 < kend;
      if (a_vec && arow && quad) {
        f32x4 v;
        __builtin_memcpy(&v, pa + kq, sizeof v);
#pragma unroll
        for (int c = 0; c < 4; ++c) av[s][c] = v[c];
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) av[s][c] = kq + c < kend ? (arow ? pa[(int64_t)(kq + c) * sak] : aone) : 0.0f;
      }
      if (b_vec && bcol && quad) {
        f32x4 v;
        __builtin_memcpy(&v, pb + kq, sizeof v);
#pragma unroll
        for (int c = 0; c < 4; ++c) bv[s][c] = v[c];
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) bv[s][c] = (kq + c < kend && bcol) ? pb[(int64_t)(kq + c) * sbk] : 0.0f;
      }
    }
  };
  constexpr int kSpan = 8 * kWsChunk;
  if (kbeg < kend) load(kbeg, a, b);
  for (int k0 = kbeg; k0 < kend; k0 += kSpan) {
    if (k0 + kSpan < kend) load(k0 + kSpan, an, bn);
#pragma unroll
    for (int s = 0; s < kWsChunk; ++s) {
      if (k0 + 8 * s >= kend) break;                // wave-uniform
#pragma unroll
      for (int c = 0; c < 4; ++c) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[s][c], b[s][c], acc, 0, 0, 0);
    }
#pragma unroll
    for (int s = 0; s < kWsChunk; ++s)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        a[s][c] = an[s][c];
        b[s][c] = bn[s][c];
      }
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) red[wave][r][lane] = acc[r];
  __syncthreads();
  for (int e = tid; e < 16 * 64; e += W * 64) {
    const int r = e >> 6, l = e & 63;
    float v = 0.0f;
#pragma unroll
    for (int w = 0; w < W; ++w) v += red[w][r][l];
    const int i = i0 + 8 * (r >> 2) + 4 * (l >> 5) + (r & 3);
    const int j = j0 + (l & 31);
    if (j >= N) continue;
    if (i < M) {
      if (EPI == kEpiBias || EPI == kEpiBiasRelu) v += bias[j];
      if (EPI == kEpiBiasRelu) v = v > 0.0f ? v : 0.0f;
      if (EPI == kEpiMask) v = mask[(int64_t)i * ldm + j] > 0.0f ? v : 0.0f;
      C[(int64_t)i * ldc + j] = v;
    } else if (i == M && ones_row) {
      ones_row[j] = v;
    }
  }
}

// Weight-gradient products C = A^T B over a long k (the mini-batch), both
// operands stored k-major: A(i, k) = A[k lda + i], B(k, j) = B[k ldb + j];
// with ones_row, row M of A is all ones and row M of the product (the column
// sums of B, the bias gradient) goes to ones_row.  Read one float per lane
// and k, as the k-split kernel must for such operands, the loads are bound
// by the compute unit's vector-memory issue rate; here each wave stages its
// k-range 32 k at a time into its own LDS slabs with 16-byte loads (8 lanes
// per k row, the next chunk's loads in flight meanwhile) and feeds the
// MFMAs from LDS in the k-split kernel's lane layout.  A workgroup of
// kWgWaves waves owns a 32 x 32 tile; the waves' partial tiles are added in
// LDS in wave order.
constexpr int kWgWaves = 16, kWgChunk = 32, kWgPad = 33;
struct WgradProblem {
  int M, N, K, kw, tiles_x;
  const float* A;
  int64_t lda;
  const float* B;
  int64_t ldb;
  float* C;
  int ldc;
  float* ones_row;
  // A training step: the tensors that C is the gradient of, and those of ones_row.
  float *w, *m, *v, *bw, *bm, *bv;
};
struct AdamStep {
  float lr, beta1, beta2, eps, c1, c2;   // c1 = 1 / (1 - beta1^t), c2 = 1 / (1 - beta2^t)
};
// Up to three products in one launch (the backward's three weight gradients
// share K): problem q owns workgroups [start[q], start[q + 1]).  step: each
// gradient element also takes its Adam step where it is produced (no product
// of the launch reads the weights), and one more workgroup stores the loss,
// the mean of (Y - T)^2 over `count` values.
struct WgradSet {
  int n;
  int start[4];
  WgradProblem p[3];
  bool step;
  AdamStep a;
  const float *Y, *T;
  int64_t count;
  float* loss;
};

// One Adam step of one parameter.
__device__ __forceinline__ void adam_update(const AdamStep& a, float gi, float* p, float* m, float* v) {
  const float mi = a.beta1 * *m + (1.0f - a.beta1) * gi;
  const float vi = a.beta2 * *v + (1.0f - a.beta2) * gi * gi;
  *m = mi;
  *v = vi;
  const float mh = mi * a.c1;
  const float vh = vi * a.c2;
  *p = *p - a.lr * mh / (__builtin_sqrtf(vh) + a.eps);
}

// out[0] = mean of (Y - T)^2 over count values by one workgroup of 1024
// threads: thread t sums elements t, t + 1024, ... (eight loads in flight
// at a time), then the waves' sums, then the 16 wave totals in order.
__device__ __forceinline__ void mse_body(const float* __restrict__ Y, const float* __restrict__ T, int64_t count,
                                         float* __restrict__ out, float* red) {
  constexpr int kU = 8;
  const int tid = threadIdx.x;
  float s = 0.0f;
  for (int64_t base = 0; base < count; base += 1024 * kU) {
    float d[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int64_t i = base + (int64_t)u * 1024 + tid;
      d[u] = i < count ? Y[i] - T[i] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) s += d[u] * d[u];
  }
  s = wave_sum_f32(s);
  if ((tid & 63) == 0) red[tid >> 6] = s;
  __syncthreads();
  if (tid == 0) {
    float t = 0.0f;
    for (int w = 0; w < 16; ++w) t += red[w];
    out[0] = t / (float)count;
  }
}

template <bool STEP>
__device__ __forceinline__ void wgrad_tile(const WgradProblem& P, const AdamStep& step, int bx, int by) {
  __shared__ float stage[kWgWaves][2][kWgChunk][kWgPad];
  static_assert(sizeof(stage) >= sizeof(float) * kWgWaves * 16 * 64, "reduction area");
  float (*red)[16][64] = reinterpret_cast<float (*)[16][64]>(&stage[0][0][0][0]);
  const int M = P.M, N = P.N, K = P.K, kw = P.kw;
  const float* __restrict__ A = P.A;
  const float* __restrict__ B = P.B;
  const int64_t lda = P.lda, ldb = P.ldb;
  float* ones_row = P.ones_row;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int g = lane >> 5;
  const int i0 = by * kWsTile, j0 = bx * kWsTile;
  const int kbeg = wave * kw;
  const int kend = (K - kbeg) < kw ? K : kbeg + kw;
  const int lr = lane >> 3, lc = 4 * (lane & 7);     // loader: rows lr + 8 q, columns lc .. lc + 3
  float ra[4][4], rb[4][4];
  auto gload = [&](int k0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int kk = k0 + 8 * q + lr;
      const bool krow = kk < kend;
      const int ia = i0 + lc, jb = j0 + lc;
      if (krow && ia + 3 < M) {
        f32x4 v;
        __builtin_memcpy(&v, A + (int64_t)kk * lda + ia, sizeof v);
#pragma unroll
        for (int e = 0; e < 4; ++e) ra[q][e] = v[e];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          ra[q][e] = !krow ? 0.0f : (ia + e < M ? A[(int64_t)kk * lda + ia + e] : (ones_row && ia + e == M ? 1.0f : 0.0f));
      }
      if (krow && jb + 3 < N) {
        f32x4 v;
        __builtin_memcpy(&v, B + (int64_t)kk * ldb + jb, sizeof v);
#pragma unroll
        for (int e = 0; e < 4; ++e) rb[q][e] = v[e];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) rb[q][e] = (krow && jb + e < N) ? B[(int64_t)kk * ldb + jb + e] : 0.0f;
      }
    }
  };
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
  if (kbeg < kend) gload(kbeg);
  for (int k0 = kbeg; k0 < kend; k0 += kWgChunk) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        stage[wave][0][8 * q + lr][lc + e] = ra[q][e];
        stage[wave][1][8 * q + lr][lc + e] = rb[q][e];
      }
    // The slabs are this wave's own: order its lanes' writes before their reads.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (k0 + kWgChunk < kend) gload(k0 + kWgChunk);
#pragma unroll
    for (int s = 0; s < kWgChunk / 8; ++s)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int kk = 8 * s + 4 * g + c;
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(stage[wave][0][kk][lane & 31], stage[wave][1][kk][lane & 31],
                                                   acc, 0, 0, 0);
      }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  __syncthreads();                                   // every wave is done with the slabs
#pragma unroll
  for (int r = 0; r < 16; ++r) red[wave][r][lane] = acc[r];
  __syncthreads();
  for (int e = tid; e < 16 * 64; e += kWgWaves * 64) {
    const int r = e >> 6, l = e & 63;
    float v = 0.0f;
#pragma unroll
    for (int w = 0; w < kWgWaves; ++w) v += red[w][r][l];
    const int i = i0 + 8 * (r >> 2) + 4 * (l >> 5) + (r & 3);
    const int j = j0 + (l & 31);
    if (j >= N) continue;
    if (i < M) {
      const int64_t e2 = (int64_t)i * P.ldc + j;
      P.C[e2] = v;
      if (STEP) adam_update(step, v, P.w + e2, P.m + e2, P.v + e2);
    } else if (i == M && ones_row) {
      ones_row[j] = v;
      if (STEP) adam_update(step, v, P.bw + j, P.bm + j, P.bv + j);
    }
  }
}

template <bool STEP>
__global__ __launch_bounds__(kWgWaves * 64) void k_gemm_wgrad(WgradSet s) {
  static_assert(kWgWaves * 64 == 1024, "mse_body");
  int b = (int)blockIdx.x;
  if constexpr (STEP) {
    __shared__ float red[16];
    if (b == 0) {
      mse_body(s.Y, s.T, s.count, s.loss, red);
      return;
    }
    --b;
  }
  int q = 0;
  while (q + 1 < s.n && b >= s.start[q + 1]) ++q;
  const int t = b - s.start[q];
  wgrad_tile<STEP>(s.p[q], s.a, t % s.p[q].tiles_x, t / s.p[q].tiles_x);
}

// Adds C = A^T B (+ ones row) to a set, both operands k-major.
static void wgrad_add(WgradSet& s, int M, int N, int K, const float* A, int64_t lda, const float* B, int64_t ldb,
                      float* C, int ldc, float* ones_row) {
  WgradProblem& P = s.p[s.n];
  const int MA = ones_row ? M + 1 : M;
  P.M = M; P.N = N; P.K = K;
  P.kw = ((K + kWgWaves - 1) / kWgWaves + kWgChunk - 1) / kWgChunk * kWgChunk;
  P.tiles_x = (N + kWsTile - 1) / kWsTile;
  P.A = A; P.lda = lda; P.B = B; P.ldb = ldb; P.C = C; P.ldc = ldc; P.ones_row = ones_row;
  if (s.n == 0) s.start[0] = 0;
  s.start[s.n + 1] = s.start[s.n] + P.tiles_x * ((MA + kWsTile - 1) / kWsTile);
  ++s.n;
}

static hipError_t wgrad_launch(const WgradSet& s, hipStream_t st) {
  if (s.n == 0 || s.start[s.n] == 0) return hipSuccess;
  if (s.step) hipLaunchKernelGGL(k_gemm_wgrad<true>, dim3(s.start[s.n] + 1), dim3(kWgWaves * 64), 0, st, s);
  else hipLaunchKernelGGL(k_gemm_wgrad<false>, dim3(s.start[s.n]), dim3(kWgWaves * 64), 0, st, s);
  return hipGetLastError();
}

// What a lane of row_dz2 reads, ahead of the dot products it waits for (1024 rows: 0.5 us
// of a step): the output weights and the hidden values of its
// columns 4 l .. 4 l + 3.
struct Dz2In {
  float w[4 * kMlpOut];
  f32x4 h;
};
__device__ __forceinline__ void load_dz2(Dz2In& in, const float* __restrict__ W3, const float* __restrict__ h2) {
  static_assert(kMlpHid == 4 * kWave, "four columns per lane");
  const int j0 = 4 * (threadIdx.x & (kWave - 1));
  __builtin_memcpy(in.w, W3 + j0 * kMlpOut, sizeof in.w);
  __builtin_memcpy(&in.h, h2 + j0, sizeof in.h);
}

// Row i of dZ2 = (dY W3^T) * (H2 > 0) by one wave, lane l taking columns 4 l ..
// 4 l + 3: six fused multiply-adds each, in the order of the outputs (relative
// error against 64 bits 4.7e-8; with each product rounded by itself 5.5e-8, and
// as a K = 6 product on the matrix cores 4.7 to 5.0e-8).
__device__ __forceinline__ void row_dz2(const float (&dy)[kMlpOut], const Dz2In& in, float* __restrict__ dz2) {
  f32x4 z;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    float t = 0.0f;
#pragma unroll
    for (int o = 0; o < kMlpOut; ++o) t = __builtin_fmaf(dy[o], in.w[c * kMlpOut + o], t);
    z[c] = in.h[c] > 0.0f ? t : 0.0f;
  }
  __builtin_memcpy(dz2 + 4 * (threadIdx.x & (kWave - 1)), &z, sizeof z);
}

// The network's output layer, Y = H2 W3 + b3, one wave per row.  With T
// (training), also the loss gradient dY = 2 (Y - T) / (M * 6), the same
// expression k_out_grad evaluates, and the second hidden layer's dZ2.  With
// idx, row i's target is row idx[i] of the table T, and that row of T and of
// the inputs X is also stored, to tb and xb: here, where the copies wait for
// nothing, and not in the product that reads the rows (they took it from 12 to
// 16 us at 1024 rows).
__global__ __launch_bounds__(256) void k_out_layer(int M, const float* __restrict__ H2, const float* __restrict__ W3,
                                                   const float* __restrict__ b3, float* __restrict__ Y,
                                                   const float* __restrict__ T, float* __restrict__ dY,
                                                   float* __restrict__ dZ2, const int32_t* __restrict__ idx,
                                                   const float* __restrict__ X, float* __restrict__ xb,
                                                   float* __restrict__ tb) {
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= M) return;                                    // whole waves
  float t[kMlpOut];
  Dz2In in;
  if (T) {
    if (dZ2) load_dz2(in, W3, H2 + (int64_t)i * kMlpHid);
    const int64_t row = idx ? idx[i] : i;
#pragma unroll
    for (int o = 0; o < kMlpOut; ++o) t[o] = T[row * kMlpOut + o];
    if (idx) {
      constexpr int kPer = kMlpIn / kWave;
      float x[kPer];
#pragma unroll
      for (int q = 0; q < kPer; ++q) x[q] = X[row * kMlpIn + q * kWave + (threadIdx.x & (kWave - 1))];
#pragma unroll
      for (int q = 0; q < kPer; ++q) xb[(int64_t)i * kMlpIn + q * kWave + (threadIdx.x & (kWave - 1))] = x[q];
    }
  }
  float acc[kMlpOut];
  wave_row_dot<kMlpOut>(H2 + (int64_t)i * kMlpHid, W3, b3, kMlpHid, kMlpOut, acc);
  const float count = (float)((int64_t)M * kMlpOut);
  float dy[kMlpOut];
  const bool first = (threadIdx.x & 63) == 0;
#pragma unroll
  for (int o = 0; o < kMlpOut; ++o) {
    const int64_t e = (int64_t)i * kMlpOut + o;
    if (first) Y[e] = acc[o];
    if (T) {
      dy[o] = 2.0f * (acc[o] - t[o]) / count;
      if (first) dY[e] = dy[o];
      if (first && idx) tb[e] = t[o];
    }
  }
  if (T && dZ2) row_dz2(dy, in, dZ2 + (int64_t)i * kMlpHid);
}

// dY = 2 (Y - T) / (M * 6) and dZ2 from stored outputs, one wave per row.
__global__ __launch_bounds__(256) void k_out_grad(int M, const float* __restrict__ Y, const float* __restrict__ T,
                                                  const float* __restrict__ W3, const float* __restrict__ H2,
                                                  float* __restrict__ dY, float* __restrict__ dZ2) {
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= M) return;
  const float count = (float)((int64_t)M * kMlpOut);
  Dz2In in;
  load_dz2(in, W3, H2 + (int64_t)i * kMlpHid);
  float dy[kMlpOut];
#pragma unroll
  for (int o = 0; o < kMlpOut; ++o) {
    const int64_t e = (int64_t)i * kMlpOut + o;
    dy[o] = 2.0f * (Y[e] - T[e]) / count;
    if ((threadIdx.x & 63) == 0) dY[e] = dy[o];
  }
  row_dz2(dy, in, dZ2 + (int64_t)i * kMlpHid);
}

template <int EPI>
static hipError_t gemm(int M, int N, int K, const float* A, int64_t sai, int64_t sak, const float* B, int64_t sbk,
                       int64_t sbj, float* C, int ldc, const float* bias, const float* mask, int ldm, hipStream_t st,
                       float* ones_row = nullptr, const int32_t* idx = nullptr) {
  if (M <= 0 || N <= 0) return hipSuccess;
  const int MA = ones_row ? M + 1 : M;
  if (MA <= kWsMaxRows) {
    const dim3 g2((N + kWsTile - 1) / kWsTile, (MA + kWsTile - 1) / kWsTile);
    if (EPI == kEpiNone && sai == 1 && sbj == 1 && K >= 256) {   // weight gradients: both operands k-major
      WgradSet set{};
      wgrad_add(set, M, N, K, A, sak, B, sbk, C, ldc, ones_row);
      return wgrad_launch(set, st);
    }
    if (K >= 512) {            // long sums: 16 waves share k
      const int kw = ((K + 15) / 16 + 7) / 8 * 8;
      hipLaunchKernelGGL((k_gemm_wsplit<EPI, 16>), g2, dim3(16 * 64), 0, st, M, N, K, kw, A, sai, sak, B, sbk, sbj,
                         C, ldc, bias, mask, ldm, ones_row, idx);
    } else {
      const int kw = ((K + 7) / 8 + 7) / 8 * 8;
      hipLaunchKernelGGL((k_gemm_wsplit<EPI, 8>), g2, dim3(8 * 64), 0, st, M, N, K, kw, A, sai, sak, B, sbk, sbj,
                         C, ldc, bias, mask, ldm, ones_row, idx);
    }
    return hipGetLastError();
  }
  const dim3 grid((N + kGemmTile - 1) / kGemmTile, (MA + kGemmTile - 1) / kGemmTile);
  hipLaunchKernelGGL((k_gemm<EPI>), grid, dim3(256), 0, st, M, N, K, A, sai, sak, B, sbk, sbj, C, ldc, bias, mask,
                     ldm, ones_row);
  return hipGetLastError();
}

__global__ __launch_bounds__(1024) void k_mse(const float* __restrict__ Y, const float* __restrict__ T,
                                              int64_t count, float* __restrict__ out) {
  __shared__ float red[16];
  mse_body(Y, T, count, out, red);
}

// The six tensors of one network as one index space for a single Adam launch.
struct AdamSet {
  float* p[6];
  const float* g[6];
  float* m[6];
  float* v[6];
  int64_t start[7];   // element e of the set is element e - start[t] of tensor t
};

// One Adam step over every parameter of the network.
__global__ __launch_bounds__(256) void k_adam(AdamSet a, AdamStep step) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= a.start[6]) return;
  int t = 0;
#pragma unroll
  for (int q = 1; q < 6; ++q) t += e >= a.start[q];
  const int64_t i = e - a.start[t];
  adam_update(step, a.g[t][i], a.p[t] + i, a.m[t] + i, a.v[t] + i);
}

// The rows idx[r] of two tables at once (a mini-batch's inputs and targets):
// elements [0, n la) of the grid copy rows of a (row length la), the rest
// rows of b.
__global__ __launch_bounds__(256) void k_gather_rows2(const float* __restrict__ a, int la, float* __restrict__ da,
                                                      const float* __restrict__ b, int lb, float* __restrict__ db,
                                                      const int32_t* __restrict__ idx, int n) {
  int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t na = (int64_t)n * la;
  if (e < na) {
    const int r = (int)(e / la);
    da[e] = a[(int64_t)idx[r] * la + (e - (int64_t)r * la)];
    return;
  }
  e -= na;
  if (e >= (int64_t)n * lb) return;
  const int r = (int)(e / lb);
  db[e] = b[(int64_t)idx[r] * lb + (e - (int64_t)r * lb)];
}

// dst[r][:] = src[idx[r]][:] for r < n rows of row_len floats.
__global__ __launch_bounds__(256) void k_gather_rows(const float* __restrict__ src, int row_len,
                                                     const int32_t* __restrict__ idx, int n, float* __restrict__ dst) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= (int64_t)n * row_len) return;
  const int r = (int)(e / row_len);
  const int c = (int)(e - (int64_t)r * row_len);
  dst[e] = src[(int64_t)idx[r] * row_len + c];
}

// ----------------------------------------------------------------------------- launchers

// With idx, the rows idx[i] of the table X (n <= kWsMaxRows).
static hipError_t hidden(const float* const* w, const float* X, int n, float* H1, float* H2, hipStream_t st,
                         const int32_t* idx) {
  // w = {w1, b1, w2, b2, w3, b3}
  hipError_t e = gemm<kEpiBiasRelu>(n, kMlpHid, kMlpIn, X, kMlpIn, 1, w[0], kMlpHid, 1, H1, kMlpHid, w[1], nullptr,
                                    0, st, nullptr, idx);
  if (e == hipSuccess)
    e = gemm<kEpiBiasRelu>(n, kMlpHid, kMlpHid, H1, kMlpHid, 1, w[2], kMlpHid, 1, H2, kMlpHid, w[3], nullptr, 0, st);
  return e;
}

hipError_t mlp_hidden(const float* const* w, const float* X, int n, float* H1, float* H2, hipStream_t st) {
  return hidden(w, X, n, H1, H2, st, nullptr);
}

hipError_t mlp_forward(const float* const* w, const float* X, int n, float* H1, float* H2, float* Y, hipStream_t st) {
  hipError_t e = mlp_hidden(w, X, n, H1, H2, st);
  if (e != hipSuccess || n <= 0) return e;
  hipLaunchKernelGGL(k_out_layer, dim3((n + 3) / 4), dim3(256), 0, st, n, H2, w[4], w[5], Y, nullptr, nullptr, nullptr,
                     nullptr, nullptr, nullptr, nullptr);
  return hipGetLastError();
}

static AdamStep adam_step(int step, float lr, float beta1, float beta2, float eps) {
  return AdamStep{lr, beta1, beta2, eps, (float)(1.0 / (1.0 - pow((double)beta1, (double)step))),
                  (float)(1.0 / (1.0 - pow((double)beta2, (double)step)))};
}

// The products behind dY and dZ2; one_launch: the three weight gradients go
// together (long sums), with `set` given also the Adam step and the loss in it.
static hipError_t backward_products(const float* const* w, const float* X, const float* H1, const float* H2, int n,
                                    float* const* g, const float* dY, float* dZ1, const float* dZ2, hipStream_t st,
                                    WgradSet* set) {
  // dZ1 = (dZ2 W2^T) * (H1 > 0)
  hipError_t e =
      gemm<kEpiMask>(n, kMlpHid, kMlpHid, dZ2, kMlpHid, 1, w[2], 1, kMlpHid, dZ1, kMlpHid, nullptr, H1, kMlpHid, st);
  if (e != hipSuccess) return e;
  // dW1 = X^T dZ1, dW2 = H1^T dZ2, dW3 = H2^T dY, each with its bias gradient
  // (column sums of the second operand) as the ones row of the same product.
  if (set) {
    wgrad_add(*set, kMlpIn, kMlpHid, n, X, kMlpIn, dZ1, kMlpHid, g[0], kMlpHid, g[1]);
    wgrad_add(*set, kMlpHid, kMlpHid, n, H1, kMlpHid, dZ2, kMlpHid, g[2], kMlpHid, g[3]);
    wgrad_add(*set, kMlpHid, kMlpOut, n, H2, kMlpHid, dY, kMlpOut, g[4], kMlpOut, g[5]);
    return wgrad_launch(*set, st);
  }
  e = gemm<kEpiNone>(kMlpIn, kMlpHid, n, X, 1, kMlpIn, dZ1, kMlpHid, 1, g[0], kMlpHid, nullptr, nullptr, 0, st, g[1]);
  if (e == hipSuccess)
    e = gemm<kEpiNone>(kMlpHid, kMlpHid, n, H1, 1, kMlpHid, dZ2, kMlpHid, 1, g[2], kMlpHid, nullptr, nullptr, 0, st,
                       g[3]);
  if (e == hipSuccess)
    e = gemm<kEpiNone>(kMlpHid, kMlpOut, n, H2, 1, kMlpHid, dY, kMlpOut, 1, g[4], kMlpOut, nullptr, nullptr, 0, st,
                       g[5]);
  return e;
}

// Rows from which the three weight gradients are one launch.
static bool long_sums(int n) { return n >= 256 && kMlpIn + 1 <= kWsMaxRows; }

hipError_t mlp_backward(const float* const* w, const float* X, const float* H1, const float* H2, const float* Y,
                        const float* T, int n, float* const* g, float* dY, float* dZ1, float* dZ2, hipStream_t st) {
  if (n > 0) {
    hipLaunchKernelGGL(k_out_grad, dim3((n + 3) / 4), dim3(256), 0, st, n, Y, T, w[4], H2, dY, dZ2);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  WgradSet set{};
  return backward_products(w, X, H1, H2, n, g, dY, dZ1, dZ2, st, long_sums(n) ? &set : nullptr);
}

// One training step: the calls' sequence (gather, forward, loss gradient,
// backward, Adam, loss) in five launches.  The products gather their rows
// where mini-batches are small enough for the k-split kernel; the output layer
// also takes dY and dZ2; the weight gradients' launch the Adam step and the
// loss.  Measured on MI355X at 1024 rows: nine launches 53.5 us a step, this
// 40.2.
hipError_t mlp_train_step(float* const* w, float* const* g, float* const* m, float* const* v, const float* X,
                          const float* T, const int32_t* idx, int n, int step, float lr, float beta1, float beta2,
                          float eps, float* xb, float* tb, float* H1, float* H2, float* Y, float* dY, float* dZ1,
                          float* dZ2, float* loss, hipStream_t st) {
  const bool fused = n <= kWsMaxRows;
  hipError_t e = hipSuccess;
  if (!fused) e = gather_rows2(X, kMlpIn, xb, T, kMlpOut, tb, idx, n, st);
  if (e == hipSuccess) e = hidden(w, fused ? X : xb, n, H1, H2, st, fused ? idx : nullptr);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_out_layer, dim3((n + 3) / 4), dim3(256), 0, st, n, H2, w[4], w[5], Y, fused ? T : tb, dY, dZ2,
                     fused ? idx : nullptr, X, xb, tb);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (long_sums(n)) {
    WgradSet set{};
    set.step = true;
    set.a = adam_step(step, lr, beta1, beta2, eps);
    set.Y = Y;
    set.T = tb;
    set.count = (int64_t)n * kMlpOut;
    set.loss = loss;
    for (int q = 0; q < 3; ++q) {
      WgradProblem& P = set.p[q];
      P.w = w[2 * q]; P.m = m[2 * q]; P.v = v[2 * q];
      P.bw = w[2 * q + 1]; P.bm = m[2 * q + 1]; P.bv = v[2 * q + 1];
    }
    return backward_products(w, xb, H1, H2, n, g, dY, dZ1, dZ2, st, &set);
  }
  e = backward_products(w, xb, H1, H2, n, g, dY, dZ1, dZ2, st, nullptr);
  if (e == hipSuccess) e = mlp_adam(w, g, m, v, step, lr, beta1, beta2, eps, st);
  if (e == hipSuccess) e = mlp_mse(Y, tb, n, loss, st);
  return e;
}

hipError_t mlp_adam(float* const* w, const float* const* g, float* const* m, float* const* v, int step, float lr,
                    float beta1, float beta2, float eps, hipStream_t st) {
  const int64_t sizes[6] = {(int64_t)kMlpIn * kMlpHid, kMlpHid, (int64_t)kMlpHid * kMlpHid, kMlpHid,
                            (int64_t)kMlpHid * kMlpOut, kMlpOut};
  AdamSet a;
  a.start[0] = 0;
  for (int t = 0; t < 6; ++t) {
    a.p[t] = w[t];
    a.g[t] = g[t];
    a.m[t] = m[t];
    a.v[t] = v[t];
    a.start[t + 1] = a.start[t] + sizes[t];
  }
  hipLaunchKernelGGL(k_adam, dim3((unsigned)((a.start[6] + 255) / 256)), dim3(256), 0, st, a,
                     adam_step(step, lr, beta1, beta2, eps));
  return hipGetLastError();
}

hipError_t mlp_mse(const float* Y, const float* T, int n, float* out, hipStream_t st) {
  hipLaunchKernelGGL(k_mse, dim3(1), dim3(1024), 0, st, Y, T, (int64_t)n * kMlpOut, out);
  return hipGetLastError();
}

hipError_t gather_rows2(const float* a, int la, float* da, const float* b, int lb, float* db, const int32_t* idx, int n,
                       hipStream_t st) {
  const int64_t total = (int64_t)n * (la + lb);
  if (total <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather_rows2, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, a, la, da, b, lb, db,
                     idx, n);
  return hipGetLastError();
}

hipError_t gather_rows(const float* src, int row_len, const int32_t* idx, int n, float* dst, hipStream_t st) {
  const int64_t total = (int64_t)n * row_len;
  if (total <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather_rows, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, src, row_len, idx, n,
                     dst);
  return hipGetLastError();
}

}  // namespace rc
