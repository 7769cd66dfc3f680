// Likelihood prescreen network 11 -> 256 -> 256 -> 256 -> 1 with exact GELU.
//
// Training (forward, backward, Adam) runs in FP32 on the matrix cores: one
// kernel takes a few rows forward and their deltas back, another forms the
// weight gradients over row splits, summed in a fixed order; the FP32 master
// weights live on the device.  The FP32 forward alone runs through an LDS-tiled
// GEMM (64 x 64 tiles, 4 x 4 outputs per thread).  Inference runs the
// hidden layers on the matrix cores: BF16 weights (round-to-nearest-even,
// stored transposed so that one lane's K-run is contiguous) and BF16
// activations feed v_mfma_f32_16x16x16_bf16 with FP32 accumulation; bias and
// GELU are applied in FP32 between layers, and the 256 -> 1 output layer is an
// FP32 dot product reduced by shuffles and a fixed-order LDS combine.
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "gw_ctx.h"

namespace gw {

constexpr int kIn = 11;
constexpr int kH = 256;
constexpr int kInPad = 32;  // K of the first layer padded for the MFMA K-step of 16
constexpr int64_t OW1 = 0;
constexpr int64_t OB1 = OW1 + kIn * kH;
constexpr int64_t OW2 = OB1 + kH;
constexpr int64_t OB2 = OW2 + kH * kH;
constexpr int64_t OW3 = OB2 + kH;
constexpr int64_t OB3 = OW3 + kH * kH;
constexpr int64_t OW4 = OB3 + kH;
constexpr int64_t OB4 = OW4 + kH;
constexpr int64_t kNPar = OB4 + 1;
// BF16 copies, transposed [out][in]: layer 1 [256][32], layers 2, 3 [256][256]
constexpr int64_t QW1 = 0;
constexpr int64_t QW2 = QW1 + kH * kInPad;
constexpr int64_t QW3 = QW2 + kH * kH;
constexpr int64_t kNQ = QW3 + kH * kH;

struct MlpScale {
  float xm[kIn];
  float xs_inv[kIn];
  double ym, ys;
};

// ---------------------------------------------------------------------------
// FP32 pieces (training and the reference forward)

__device__ inline float gelu_f(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }

__device__ inline float gelu_grad_f(float z) {
  return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

__global__ void k_mlp_stdin(const double* __restrict__ x, int64_t n, MlpScale sc, float* __restrict__ xs) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * kIn) return;
  const int j = (int)(i % kIn);
  xs[i] = ((float)x[i] - sc.xm[j]) * sc.xs_inv[j];
}

// C = A B + bias (FP32 forward).
__global__ void __launch_bounds__(256) k_gemm(int M, int N, int K, const float* __restrict__ A, int lda,
                                              const float* __restrict__ B, int ldb, float* __restrict__ C, int ldc,
                                              const float* __restrict__ bias) {
  __shared__ float As[16][64 + 4];
  __shared__ float Bs[16][64 + 4];
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const int i0 = blockIdx.y * 64, j0 = blockIdx.x * 64;
  float acc[4][4];
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[r][c] = 0.0f;
  for (int k0 = 0; k0 < K; k0 += 16) {
    for (int e = threadIdx.x; e < 1024; e += 256) {
      const int ii = e >> 4, kk = e & 15;
      const int gi = i0 + ii, gk = k0 + kk;
      As[kk][ii] = gi < M && gk < K ? A[(int64_t)gi * lda + gk] : 0.0f;
    }
    for (int e = threadIdx.x; e < 1024; e += 256) {
      const int kk = e >> 6, jj = e & 63;
      const int gj = j0 + jj, gk = k0 + kk;
      Bs[kk][jj] = gj < N && gk < K ? B[(int64_t)gk * ldb + gj] : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) a[r] = As[kk][ty * 4 + r];
#pragma unroll
      for (int c = 0; c < 4; ++c) b[c] = Bs[kk][tx * 4 + c];
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[r][c] = fmaf(a[r], b[c], acc[r][c]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = i0 + ty * 4 + r;
    if (i >= M) continue;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int j = j0 + tx * 4 + c;
      if (j < N) C[(int64_t)i * ldc + j] = acc[r][c] + bias[j];
    }
  }
}

__global__ void k_gelu_fwd(const float* __restrict__ z, float* __restrict__ a, int64_t count) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < count) a[e] = gelu_f(z[e]);
}

// ---------------------------------------------------------------------------
// Loss and gradient of a batch, FP32 on the matrix cores, in four launches.
// Bound by latency and by the weights each workgroup reads from L2.  1024 rows:
// 26 us forward and deltas, 13 weight gradients, 4 each for the transposes and
// the sum over splits; 440 us as 28 launches of a vector-ALU GEMM of 64 x 64
// tiles (16 to 64 workgroups each), elementwise kernels and column sums.

typedef float f4v __attribute__((ext_vector_type(4)));

// W2 and W3 transposed, for the backward products (32 x 32 tiles).
__global__ void __launch_bounds__(256) k_transpose(const float* __restrict__ p, float* __restrict__ t) {
  __shared__ float tile[32][33];
  const float* __restrict__ src = p + (blockIdx.z == 0 ? OW2 : OW3);
  float* __restrict__ dst = t + (int64_t)blockIdx.z * kH * kH;
  const int x = threadIdx.x & 31, y = threadIdx.x >> 5, i0 = blockIdx.y * 32, j0 = blockIdx.x * 32;
  for (int r = y; r < 32; r += 8) tile[r][x] = src[(i0 + r) * kH + j0 + x];
  __syncthreads();
  for (int r = y; r < 32; r += 8) dst[(j0 + r) * kH + i0 + x] = tile[x][r];
}

// Batch state between the launches: inputs [n][16] (standardised, zero
// beyond kIn), activations and deltas of the hidden layers [n][kH] each, per
// row dy and (y - t)^2.
struct TrainView {
  float *xs, *a1, *a2, *a3, *d1, *d2, *d3, *dy, *r2;
};

// The 4 R rows of a workgroup against 64 features per wave: lane = feature,
// acc[r][q] of row 4 r + q over the kH inputs of act (LDS, [4 R][kH + 4]) and
// w [kH][kH], by
// the 4x4x1 matrix instruction (16 blocks of 4 rows x 4 features at one k; the
// rows are the same in every block, so 4-row tiles keep all of its rate and
// 1024 rows fill the 256 CUs).  Weights are read ahead, 64 k of them with few
// rows (1024 rows: 26 us for k_train_rows, 34 at 16 k).
template <int R>
__device__ inline void rows_times(const float* __restrict__ act, const float* __restrict__ w, int j, f4v acc[R]) {
  constexpr int kStride = kH + 4, kStep = R == 1 ? 64 : 16;
  f4v part[R][4];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int q = 0; q < 4; ++q) part[r][q] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
  const float* __restrict__ row = act + (threadIdx.x & 3) * kStride;
  float cur[kStep], nxt[kStep];
#pragma unroll
  for (int k = 0; k < kStep; ++k) cur[k] = w[(int64_t)k * kH + j];
#pragma unroll
  for (int k0 = 0; k0 < kH; k0 += kStep) {
    const int kn = k0 + kStep < kH ? k0 + kStep : k0;
#pragma unroll
    for (int k = 0; k < kStep; ++k) nxt[k] = w[(int64_t)(kn + k) * kH + j];
#pragma unroll
    for (int k = 0; k < kStep; k += 4)
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const f4v a = *(const f4v*)(row + 4 * r * kStride + k0 + k);
#pragma unroll
        for (int q = 0; q < 4; ++q)
          part[r][q] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[q], cur[k + q], part[r][q], 0, 0, 0);
      }
#pragma unroll
    for (int k = 0; k < kStep; ++k) cur[k] = nxt[k];
  }
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] = (part[r][0] + part[r][1]) + (part[r][2] + part[r][3]);
}

// Forward and the deltas backward of 4 R rows per workgroup (wave = 64
// features).  wt: W2, W3 transposed.
template <int R>
__global__ void __launch_bounds__(256) k_train_rows(const double* __restrict__ x, const double* __restrict__ target,
                                                    int64_t n, MlpScale sc, const float* __restrict__ p,
                                                    const float* __restrict__ wt, TrainView v) {
  constexpr int kRows = 4 * R, kStride = kH + 4;
  __shared__ __align__(16) float act[2][kRows * kStride];
  __shared__ float ysum[4][kRows];
  __shared__ float dys[kRows];
  const int j = threadIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t i0 = (int64_t)blockIdx.x * kRows;
  for (int e = threadIdx.x; e < kRows * 16; e += 256) {
    const int r = e >> 4, k = e & 15;
    const int64_t i = i0 + r;
    const float f = i < n && k < kIn ? ((float)x[i * kIn + k] - sc.xm[k]) * sc.xs_inv[k] : 0.0f;
    act[0][r * kStride + k] = f;
    if (i < n) v.xs[i * 16 + k] = f;
  }
  __syncthreads();
  f4v acc[R], z1[R], z2[R], z3[R];
  // out = GELU(acc + b) to the next activation buffer and to memory
  auto layer = [&](int from, float b, f4v* z, float* __restrict__ out) {
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        z[r][q] = acc[r][q] + b;
        const float a = gelu_f(z[r][q]);
        const int row = 4 * r + q;
        act[from ^ 1][row * kStride + j] = a;
        if (i0 + row < n) out[(i0 + row) * kH + j] = a;
        acc[r][q] = a;
      }
    __syncthreads();
  };
  {  // K = 11: the weights of the padding are zero by the input alone
    f4v s[R];
#pragma unroll
    for (int r = 0; r < R; ++r) s[r] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
    const float* __restrict__ row = act[0] + (threadIdx.x & 3) * kStride;
#pragma unroll
    for (int k = 0; k < kIn; ++k) {
      const float w = p[OW1 + k * kH + j];
#pragma unroll
      for (int r = 0; r < R; ++r)
        s[r] = __builtin_amdgcn_mfma_f32_4x4x1f32(row[4 * r * kStride + k], w, s[r], 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = s[r];
  }
  layer(0, p[OB1 + j], z1, v.a1);
  rows_times<R>(act[1], p + OW2, j, acc);
  layer(1, p[OB2 + j], z2, v.a2);
  rows_times<R>(act[0], p + OW3, j, acc);
  layer(0, p[OB3 + j], z3, v.a3);
  // output, loss terms and dy: lanes, then waves, in a fixed order
  const float w4 = p[OW4 + j];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float t = acc[r][q] * w4;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
      if (lane == 0) ysum[wave][4 * r + q] = t;
    }
  __syncthreads();
  if (threadIdx.x < kRows) {
    const int64_t i = i0 + threadIdx.x;
    const int r = threadIdx.x;
    float d = 0.0f;
    if (i < n) {
      const float y = ((ysum[0][r] + ysum[1][r]) + (ysum[2][r] + ysum[3][r])) + p[OB4];
      const float e = y - (float)((target[i] - sc.ym) * (1.0 / sc.ys));
      d = 2.0f * e / (float)n;
      v.dy[i] = d;
      v.r2[i] = e * e;
    }
    dys[r] = d;
  }
  __syncthreads();
  auto delta = [&](int to, const f4v* z, float* __restrict__ out) {
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row = 4 * r + q;
        const float d = acc[r][q] * gelu_grad_f(z[r][q]);
        act[to][row * kStride + j] = d;
        if (i0 + row < n) out[(i0 + row) * kH + j] = d;
      }
    __syncthreads();
  };
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[r][q] = dys[4 * r + q] * w4;
  delta(0, z3, v.d3);
  rows_times<R>(act[0], wt + kH * kH, j, acc);
  delta(1, z2, v.d2);
  rows_times<R>(act[1], wt, j, acc);
  delta(0, z1, v.d1);
}

// Weight gradients over the rows of split blockIdx.y, into part [split]
// [kNPar + 1] (the last: the loss sum): one workgroup per 64 x 64 tile of dW3
// and dW2 (32), per 64 columns of dW1 (4) and per 64 rows of dW4 (4).  A wave
// takes a quarter of the split's rows; the 16x16x4 matrix instruction has the
// rows as its k.  A lane's 16-byte read holds one value of four tiles: tile a
// has the features 4 c + a, c < 16.  The tiles of dW3, dW2 at i0 = 0 and those of
// dW1 carry the column sums of the deltas (the bias gradients) along.
__global__ void __launch_bounds__(256) k_train_weights(int64_t n, int rows_per, TrainView v, float* __restrict__ part) {
  __shared__ float red[3][64][65];
  __shared__ float cred[3][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c = lane & 15, g = lane >> 4;
  const int64_t s0 = (int64_t)blockIdx.y * rows_per;
  const int64_t s1 = s0 + rows_per < n ? s0 + rows_per : n;
  const int quarter = rows_per / 4;  // a multiple of 4
  const int64_t r0 = s0 + wave * quarter < s1 ? s0 + wave * quarter : s1;
  const int64_t r1 = r0 + quarter < s1 ? r0 + quarter : s1;
  float* __restrict__ out = part + (int64_t)blockIdx.y * (kNPar + 1);
  const int t = blockIdx.x;
  f4v col = {0.0f, 0.0f, 0.0f, 0.0f};  // column sums of this lane's rows
  // (wave 0 + wave 1) + wave 2 + wave 3, lanes by their row group first
  auto group_sum = [&](f4v s) {
#pragma unroll
    for (int o = 16; o < 64; o <<= 1)
#pragma unroll
      for (int q = 0; q < 4; ++q) s[q] += __shfl_xor(s[q], o, 64);
    return s;
  };
  if (t < 36) {
    const bool first = t >= 32;
    const int m = t >> 4, i0 = first ? 0 : 64 * ((t >> 2) & 3), j0 = 64 * (t & 3);
    const float* __restrict__ A = first ? v.xs : (m == 0 ? v.a2 : v.a1);
    const float* __restrict__ D = first ? v.d1 : (m == 0 ? v.d3 : v.d2);
    const int lda = first ? 16 : kH;
    f4v acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) acc[a][b] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
    const f4v zero = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
    for (int64_t r = r0; r < r1; r += 4) {
      const int64_t i = r + g;
      f4v av = zero, dv = zero;
      if (i < r1) {
        dv = *(const f4v*)(D + i * kH + j0 + 4 * c);
        if (first)
          av[0] = A[i * 16 + c];
        else
          av = *(const f4v*)(A + i * (int64_t)lda + i0 + 4 * c);
      }
      col += dv;
      if (first) {
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[0][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[0], dv[b], acc[0][b], 0, 0, 0);
      } else {
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int b = 0; b < 4; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[a], dv[b], acc[a][b], 0, 0, 0);
      }
    }
    // tile (a, b): register q of this lane is row 4 g + q, column c; feature
    // 4 row + a (the first layer: row), 4 c + b
    col = group_sum(col);
    if (wave > 0) {
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (!first || a == 0) red[wave - 1][first ? 4 * g + q : 4 * (4 * g + q) + a][4 * c + b] = acc[a][b][q];
      if (g == 0)
#pragma unroll
        for (int b = 0; b < 4; ++b) cred[wave - 1][4 * c + b] = col[b];
    }
    __syncthreads();
    if (wave > 0) return;
    float* __restrict__ W = out + (first ? OW1 : (m == 0 ? OW3 : OW2));
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int fi = first ? 4 * g + q : 4 * (4 * g + q) + a;
        if (first && (a > 0 || fi >= kIn)) continue;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const int fj = 4 * c + b;
          W[(int64_t)(i0 + fi) * kH + j0 + fj] =
              ((acc[a][b][q] + red[0][fi][fj]) + red[1][fi][fj]) + red[2][fi][fj];
        }
      }
    if ((first || i0 == 0) && g == 0) {
      float* __restrict__ B = out + (first ? OB1 : (m == 0 ? OB3 : OB2));
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int fj = 4 * c + b;
        B[j0 + fj] = ((col[b] + cred[0][fj]) + cred[1][fj]) + cred[2][fj];
      }
    }
    return;
  }
  const int j0 = 64 * (t - 36);
  float sd = 0.0f, sr = 0.0f;
  for (int64_t r = r0; r < r1; r += 4) {
    const int64_t i = r + g;
    if (i < r1) {
      const float d = v.dy[i];
      const f4v a = *(const f4v*)(v.a3 + i * kH + j0 + 4 * c);
      col += a * d;
      sd += d;
      sr += v.r2[i];
    }
  }
  col = group_sum(col);
  const f4v e = group_sum(f4v{sd, sr, 0.0f, 0.0f});
  if (wave > 0 && g == 0) {
#pragma unroll
    for (int b = 0; b < 4; ++b) cred[wave - 1][4 * c + b] = col[b];
    red[wave - 1][0][0] = e[0];
    red[wave - 1][0][1] = e[1];
  }
  __syncthreads();
  if (wave > 0 || g > 0) return;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int fj = 4 * c + b;
    out[OW4 + j0 + fj] = ((col[b] + cred[0][fj]) + cred[1][fj]) + cred[2][fj];
  }
  if (j0 == 0 && c == 0) {
    out[OB4] = ((e[0] + red[0][0][0]) + red[1][0][0]) + red[2][0][0];
    out[kNPar] = ((e[1] + red[0][0][1]) + red[1][0][1]) + red[2][0][1];
  }
}

// g = sum of the splits in order; the loss is the mean of its terms.
__global__ void __launch_bounds__(256) k_train_sum(const float* __restrict__ part, int splits, int64_t n,
                                                   float* __restrict__ g, float* __restrict__ loss) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e > kNPar) return;
  float s = 0.0f;
#pragma unroll 8
  for (int z = 0; z < splits; ++z) s += part[(int64_t)z * (kNPar + 1) + e];
  if (e < kNPar)
    g[e] = s;
  else
    *loss = s / (float)n;
}

__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m, float* __restrict__ v,
                       int64_t count, float lr, float c1, float c2) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= count) return;
  const float gg = g[e];
  const float mm = 0.9f * m[e] + 0.1f * gg;
  const float vv = 0.999f * v[e] + 0.001f * gg * gg;
  m[e] = mm;
  v[e] = vv;
  p[e] -= lr * (mm * c1) / (sqrtf(vv * c2) + 1e-8f);
}

__device__ inline uint16_t to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// BF16 transposed copies of W1 (K padded to 32 with zeros), W2, W3.
__global__ void k_to_bf16(const float* __restrict__ p, uint16_t* __restrict__ q) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= kNQ) return;
  if (e < QW2) {
    const int o = (int)(e / kInPad), k = (int)(e % kInPad);
    q[e] = k < kIn ? to_bf16(p[OW1 + (int64_t)k * kH + o]) : 0;
  } else {
    const int64_t base = e < QW3 ? OW2 : OW3;
    const int64_t r = e - (e < QW3 ? QW2 : QW3);
    const int o = (int)(r / kH), k = (int)(r % kH);
    q[e] = to_bf16(p[base + (int64_t)k * kH + o]);
  }
}

// ---------------------------------------------------------------------------
// BF16 MFMA inference: one workgroup (8 waves) per 32 RT rows.  Each layer is
// computed transposed, out^T [feature][row] = W [feature][k] act^T [k][row],
// with the 16x16x32 BF16 matrix instruction (FP32 accumulation): operand A is
// a 16-feature x 32-k tile of the weights (read from memory, one k-step
// ahead), operand B a 32-k x 16-row tile of the activations (LDS, rows of
// kActStride bf16 so that the 16 rows of a read fall in distinct banks); a
// lane's 4 results are 4 consecutive features of one row, stored as one
// 8-byte write.  Wave w owns features 64 (w mod 4) .. + 63 of rows
// 16 RT (w / 4) .. + 16 RT - 1: 4 feature tiles x RT row tiles.

typedef short s8v __attribute__((ext_vector_type(8)));

constexpr int kActStride = kH + 8;  // bf16 per activation row in LDS

__device__ inline f4v mfma_bf16_16x16x32(s8v a, s8v b, f4v c) {
  typedef __bf16 b8v __attribute__((ext_vector_type(8)));
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8v, a), __builtin_bit_cast(b8v, b), c, 0, 0,
                                                 0);
}

template <int RT>
__global__ void __launch_bounds__(512) k_mlp_infer(const double* __restrict__ x, int64_t n, MlpScale sc,
                                                   const uint16_t* __restrict__ q, const float* __restrict__ p,
                                                   double* __restrict__ out) {
  constexpr int kRows = 32 * RT;
  __shared__ __attribute__((aligned(16))) uint16_t act[kRows * kActStride];  // [row][k]
  __shared__ float red[4][kRows];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int fw = wave & 3, rw = wave >> 2;  // feature block, row half
  const int64_t r0 = (int64_t)blockIdx.x * kRows;
  // standardised input, K padded to 32
  for (int e = threadIdx.x; e < kRows * kInPad; e += 512) {
    const int row = e / kInPad, k = e % kInPad;
    float v = 0.0f;
    if (k < kIn && r0 + row < n) v = ((float)x[(r0 + row) * kIn + k] - sc.xm[k]) * sc.xs_inv[k];
    act[row * kActStride + k] = to_bf16(v);
  }
  __syncthreads();
  const int l16 = lane & 15;        // feature (A) / row (B) within a tile
  const int lk = (lane >> 4) * 8;   // this lane's 8 values of the 32-k step
  const int lf = (lane >> 4) * 4;   // first of this lane's 4 output features in a tile
  f4v acc[4][RT];                   // [feature tile][row tile]
  for (int layer = 0; layer < 3; ++layer) {
    const int K = layer == 0 ? kInPad : kH;
    const uint16_t* __restrict__ W = q + (layer == 0 ? QW1 : (layer == 1 ? QW2 : QW3));
    const float* __restrict__ bias = p + (layer == 0 ? OB1 : (layer == 1 ? OB2 : OB3));
#pragma unroll
    for (int ft = 0; ft < 4; ++ft)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) acc[ft][rt] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
    const uint16_t* __restrict__ wrow = W + (int64_t)(fw * 64 + l16) * K + lk;
    s8v a_cur[4], a_nxt[4];
#pragma unroll
    for (int ft = 0; ft < 4; ++ft) a_cur[ft] = *(const s8v*)(wrow + (int64_t)ft * 16 * K);
    for (int k0 = 0; k0 < K; k0 += 32) {
      if (k0 + 32 < K) {
#pragma unroll
        for (int ft = 0; ft < 4; ++ft) a_nxt[ft] = *(const s8v*)(wrow + (int64_t)ft * 16 * K + k0 + 32);
      }
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const s8v b = *(const s8v*)&act[((rw * RT + rt) * 16 + l16) * kActStride + k0 + lk];
#pragma unroll
        for (int ft = 0; ft < 4; ++ft) acc[ft][rt] = mfma_bf16_16x16x32(a_cur[ft], b, acc[ft][rt]);
      }
      if (k0 + 32 < K) {
#pragma unroll
        for (int ft = 0; ft < 4; ++ft) a_cur[ft] = a_nxt[ft];
      }
    }
    // bias + GELU in FP32; D[feature = lf + j][row = l16] per tile
#pragma unroll
    for (int ft = 0; ft < 4; ++ft) {
      const float4 bc = *(const float4*)&bias[fw * 64 + ft * 16 + lf];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        acc[ft][rt][0] = gelu_f(acc[ft][rt][0] + bc.x);
        acc[ft][rt][1] = gelu_f(acc[ft][rt][1] + bc.y);
        acc[ft][rt][2] = gelu_f(acc[ft][rt][2] + bc.z);
        acc[ft][rt][3] = gelu_f(acc[ft][rt][3] + bc.w);
      }
    }
    __syncthreads();  // every wave has read this layer's input
    if (layer < 2) {
#pragma unroll
      for (int ft = 0; ft < 4; ++ft)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          const uint32_t lo = (uint32_t)to_bf16(acc[ft][rt][0]) | ((uint32_t)to_bf16(acc[ft][rt][1]) << 16);
          const uint32_t hi = (uint32_t)to_bf16(acc[ft][rt][2]) | ((uint32_t)to_bf16(acc[ft][rt][3]) << 16);
          *(uint2*)&act[((rw * RT + rt) * 16 + l16) * kActStride + fw * 64 + ft * 16 + lf] = make_uint2(lo, hi);
        }
      __syncthreads();
    }
  }
  // output layer 256 -> 1 in FP32: per-lane partial over its 16 features,
  // then the 4 lane groups that share a row, then the 4 feature blocks in order
  float w4[4][4];
#pragma unroll
  for (int ft = 0; ft < 4; ++ft) {
    const float4 w = *(const float4*)&p[OW4 + fw * 64 + ft * 16 + lf];
    w4[ft][0] = w.x;
    w4[ft][1] = w.y;
    w4[ft][2] = w.z;
    w4[ft][3] = w.w;
  }
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    float v = 0.0f;
#pragma unroll
    for (int ft = 0; ft < 4; ++ft)
#pragma unroll
      for (int j = 0; j < 4; ++j) v = fmaf(acc[ft][rt][j], w4[ft][j], v);
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    if (lane < 16) red[fw][(rw * RT + rt) * 16 + l16] = v;
  }
  __syncthreads();
  if (threadIdx.x < kRows && r0 + threadIdx.x < n) {
    const int t = threadIdx.x;
    const float y = ((red[0][t] + red[1][t]) + (red[2][t] + red[3][t])) + p[OB4];
    out[r0 + t] = sc.ym + sc.ys * (double)y;
  }
}

// Prescreen decision per candidate: bit0 exact evaluation wanted, bit1 the
// prediction passes (pred >= log L* - margin), bit2 audited (a rejected
// candidate drawn for an exact check with probability audit_frac, Philox
// word 0 of counter (i, 0, 0, 0) under key (seed, 1)).
__device__ inline double audit_uniform(uint64_t seed, int64_t i) {
  const uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
  const uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
  uint64_t c[4] = {(uint64_t)i, 0ull, 0ull, 0ull};
  uint64_t k0 = seed, k1 = 1ull;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t hi0 = __umul64hi(M0, c[0]), lo0 = M0 * c[0];
    const uint64_t hi1 = __umul64hi(M1, c[2]), lo1 = M1 * c[2];
    const uint64_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
    c[0] = n0;
    c[1] = lo1;
    c[2] = n2;
    c[3] = lo0;
    k0 += W0;
    k1 += W1;
  }
  return ((double)(c[0] >> 11) + 0.5) * 1.1102230246251565404e-16;
}

__global__ void k_prescreen_flags(const double* __restrict__ pred, int64_t n, double cut, double audit_frac,
                                  uint64_t seed, int use_mlp, int32_t* __restrict__ flags) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int f;
  if (!use_mlp) {
    f = 1;
  } else if (pred[i] >= cut) {
    f = 3;
  } else {
    f = audit_uniform(seed, i) < audit_frac ? 5 : 0;
  }
  flags[i] = f;
}

// Positions of the selected rows (bit0) by a one-workgroup scan; pos[n] holds
// the count.
__global__ void __launch_bounds__(256) k_select_scan(const int32_t* __restrict__ flags, int64_t n,
                                                     int64_t* __restrict__ pos) {
  __shared__ int64_t part[256];
  const int64_t per = (n + 255) / 256;
  const int64_t b = threadIdx.x * per;
  const int64_t e = b + per < n ? b + per : n;
  int64_t s = 0;
  for (int64_t i = b; i < e; ++i) s += flags[i] & 1;
  part[threadIdx.x] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t run = 0;
    for (int j = 0; j < 256; ++j) {
      const int64_t v = part[j];
      part[j] = run;
      run += v;
    }
    pos[n] = run;
  }
  __syncthreads();
  int64_t run = part[threadIdx.x];
  for (int64_t i = b; i < e; ++i) {
    pos[i] = run;
    run += flags[i] & 1;
  }
}

__global__ void k_gather_rows(const double* __restrict__ x, int64_t n, const int32_t* __restrict__ flags,
                              const int64_t* __restrict__ pos, double* __restrict__ xs) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n || !(flags[i] & 1)) return;
  const int64_t j = pos[i];
  for (int d = 0; d < kIn; ++d) xs[j * kIn + d] = x[i * kIn + d];
}

__global__ void k_scatter_logl(const double* __restrict__ sub, int64_t n, const int32_t* __restrict__ flags,
                               const int64_t* __restrict__ pos, double* __restrict__ logl) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  logl[i] = (flags[i] & 1) ? sub[pos[i]] : -INFINITY;
}

__global__ void k_unscale(const float* __restrict__ y, int64_t n, MlpScale sc, double* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = sc.ym + sc.ys * (double)y[i];
}

}  // namespace gw

using namespace gw;

struct gw_mlp {
  gw_ctx* ctx = nullptr;
  float* p = nullptr;
  float* g = nullptr;
  float* m = nullptr;
  float* v = nullptr;
  uint16_t* q = nullptr;
  bool q_dirty = true;
  int64_t t = 0;
  MlpScale sc{};
  uint64_t sc_version = 0;  // bumped whenever sc changes (a captured launch bakes sc in)
  float* ws = nullptr;  // workspace of training and of the FP32 forward
  int64_t ws_cap = 0;
  float* loss = nullptr;  // device scalar behind g
  float* h_g = nullptr;   // pinned copy of g and the loss
  // prescreen workspace
  void* pre = nullptr;
  int64_t pre_cap = 0;
  int64_t* h_count = nullptr;  // pinned
};

namespace {

// Workspace of the FP32 forward and of training (floats).
gw_status mlp_ws(gw_mlp* m, int64_t count) {
  if (count <= m->ws_cap) return GW_OK;
  if (m->ws) (void)hipFree(m->ws);
  m->ws = nullptr;
  m->ws_cap = 0;
  gw_status s = check_hip(hipMalloc((void**)&m->ws, (size_t)count * sizeof(float)), "mlp workspace");
  if (s == GW_OK) m->ws_cap = count;
  return s;
}

inline unsigned nblk(int64_t n) { return (unsigned)((n + 255) / 256); }

// FP32 forward of ``rows`` inputs into y (workspace a: one activation buffer
// of rows kIn, then two of rows kH).
gw_status forward32(gw_mlp* m, const double* x, int64_t rows, float* y, float* a, hipStream_t st) {
  const int R = (int)rows;
  float *xs = a, *h = xs + rows * kIn, *z = h + rows * kH;
  auto gemm = [&](const float* in, int k, int64_t w, int64_t b, int cols, float* out) {
    hipLaunchKernelGGL(k_gemm, dim3((cols + 63) / 64, (R + 63) / 64), dim3(256), 0, st, R, cols, k, in, k, m->p + w,
                       cols, out, cols, m->p + b);
  };
  auto gelu = [&] {
    hipLaunchKernelGGL(k_gelu_fwd, dim3(nblk(rows * kH)), dim3(256), 0, st, z, h, rows * kH);
  };
  hipLaunchKernelGGL(k_mlp_stdin, dim3(nblk(rows * kIn)), dim3(256), 0, st, x, rows, m->sc, xs);
  gemm(xs, kIn, OW1, OB1, kH, z);
  gelu();
  gemm(h, kH, OW2, OB2, kH, z);
  gelu();
  gemm(h, kH, OW3, OB3, kH, z);
  gelu();
  gemm(h, kH, OW4, OB4, 1, y);
  return check_hip(hipGetLastError(), "mlp forward");
}

// Loss and gradients of one batch into m->g.
gw_status grad32(gw_mlp* m, const double* x, const double* y, int64_t n, hipStream_t st) {
  // rows of a split of the weight gradients: 128 up to 32 splits (1024 rows: 320
  // workgroups of 8 splits)
  const int64_t rows_per = std::max<int64_t>(128, ((n + 31) / 32 + 15) / 16 * 16);
  const int splits = (int)((n + rows_per - 1) / rows_per);
  const int64_t per_row = 16 + 6 * kH + 2, wt_n = 2 * kH * kH, np = (n + 3) / 4 * 4;
  gw_status s = mlp_ws(m, np * per_row + wt_n + (int64_t)splits * (kNPar + 1));
  if (s != GW_OK) return s;
  TrainView v;
  float* w = m->ws;
  float* wt = w;
  w += wt_n;
  v.xs = w, w += np * 16;
  for (float** q : {&v.a1, &v.a2, &v.a3, &v.d1, &v.d2, &v.d3}) *q = w, w += np * kH;
  v.dy = w, w += np;
  v.r2 = w, w += np;
  float* part = w;
  hipLaunchKernelGGL(k_transpose, dim3(kH / 32, kH / 32, 2), dim3(256), 0, st, (const float*)m->p, wt);
  auto rows = [&](auto kernel, int64_t r) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)((n + r - 1) / r)), dim3(256), 0, st, x, y, n, m->sc,
                       (const float*)m->p, (const float*)wt, v);
  };
  // rows per workgroup: 4, up to four workgroups a CU; beyond, 16 share the
  // weights' reads (3000 rows: 144 us a call of 4, 175 of 16; 8192: 215 and 200)
  if (n <= 4096)
    rows(k_train_rows<1>, 4);
  else
    rows(k_train_rows<4>, 16);
  hipLaunchKernelGGL(k_train_weights, dim3(40, (unsigned)splits), dim3(256), 0, st, n, (int)rows_per, v, part);
  hipLaunchKernelGGL(k_train_sum, dim3(nblk(kNPar + 1)), dim3(256), 0, st, (const float*)part, splits, n, m->g,
                     m->loss);
  return check_hip(hipGetLastError(), "mlp gradient");
}

uint64_t splitmix(uint64_t& s) {
  uint64_t z = (s += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

}  // namespace

namespace gw {

const gw_ctx* mlp_ctx(const gw_mlp* m) { return m->ctx; }

uint64_t mlp_scale_version(const gw_mlp* m) { return m->sc_version; }

gw_status mlp_prepare(gw_mlp* m, hipStream_t st) {
  if (!m->q_dirty) return GW_OK;
  hipLaunchKernelGGL(k_to_bf16, dim3(nblk(kNQ)), dim3(256), 0, st, m->p, m->q);
  gw_status s = check_hip(hipGetLastError(), "bf16 conversion launch");
  if (s == GW_OK) m->q_dirty = false;
  return s;
}

gw_status mlp_infer(gw_mlp* m, const double* x, int64_t n, double* out, hipStream_t st) {
  if (n == 0) return GW_OK;
  auto launch = [&](auto kernel, int64_t rows) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)((n + rows - 1) / rows)), dim3(512), 0, st, x, n, m->sc,
                       (const uint16_t*)m->q, (const float*)m->p, out);
  };
  // the fewest rows per workgroup that still is one workgroup a CU (a row's
  // result is the same in each): 25, 31 and 42 us a call of 32, 64 and 128 rows
  // up to that point; beyond it fewer rows read the weights more often (12,000
  // rows: 37 us of 32, 31 of 64; 32,768: 72, 45, 43)
  if (n <= 8192)
    launch(k_mlp_infer<1>, 32);
  else if (n <= 16384)
    launch(k_mlp_infer<2>, 64);
  else
    launch(k_mlp_infer<4>, 128);
  return check_hip(hipGetLastError(), "mlp inference launch");
}

}  // namespace gw

extern "C" {

gw_status gw_mlp_create(gw_ctx* ctx, uint64_t seed, gw_mlp** out) {
  if (!ctx || !out) return set_error(GW_EINVAL, "gw_mlp_create: null argument");
  *out = nullptr;
  gw_status s = check_hip(hipSetDevice(ctx->device), "hipSetDevice");
  if (s != GW_OK) return s;
  gw_mlp* m = new (std::nothrow) gw_mlp();
  if (!m) return set_error(GW_ENOMEM, "gw_mlp_create: host allocation");
  m->ctx = ctx;
  for (int j = 0; j < kIn; ++j) {
    m->sc.xm[j] = 0.5f;
    m->sc.xs_inv[j] = 3.4641016f;  // 1 / sqrt(1/12): standardised uniform
  }
  m->sc.ym = 0.0;
  m->sc.ys = 1.0;
  // He-normal weights from a splitmix64 stream (Box-Muller), zero biases.
  std::vector<float> h(kNPar, 0.0f);
  uint64_t st = seed;
  auto normal = [&]() {
    const double u1 = ((splitmix(st) >> 11) + 0.5) * 1.1102230246251565e-16;
    const double u2 = ((splitmix(st) >> 11) + 0.5) * 1.1102230246251565e-16;
    return sqrt(-2.0 * log(u1)) * cos(6.283185307179586 * u2);
  };
  auto fill = [&](int64_t off, int fan_in, int64_t count) {
    const double sd = sqrt(2.0 / fan_in);
    for (int64_t e = 0; e < count; ++e) h[off + e] = (float)(sd * normal());
  };
  fill(OW1, kIn, kIn * kH);
  fill(OW2, kH, kH * kH);
  fill(OW3, kH, kH * kH);
  fill(OW4, kH, kH);
  float* bufs[4] = {nullptr, nullptr, nullptr, nullptr};
  for (int i = 0; i < 4 && s == GW_OK; ++i) s = check_hip(hipMalloc((void**)&bufs[i], (kNPar + 1) * sizeof(float)), "mlp");
  if (s == GW_OK) s = check_hip(hipMalloc((void**)&m->q, kNQ * sizeof(uint16_t)), "mlp");
  m->p = bufs[0];
  m->g = bufs[1];
  m->loss = m->g + kNPar;
  m->m = bufs[2];
  m->v = bufs[3];
  if (s == GW_OK) s = check_hip(hipMemcpy(m->p, h.data(), kNPar * sizeof(float), hipMemcpyHostToDevice), "mlp copy");
  if (s == GW_OK) s = check_hip(hipMemset(m->m, 0, kNPar * sizeof(float)), "mlp memset");
  if (s == GW_OK) s = check_hip(hipMemset(m->v, 0, kNPar * sizeof(float)), "mlp memset");
  if (s == GW_OK) s = check_hip(hipMemset(m->g, 0, kNPar * sizeof(float)), "mlp memset");
  if (s != GW_OK) {
    for (float* b : bufs)
      if (b) (void)hipFree(b);
    if (m->q) (void)hipFree(m->q);
    delete m;
    return s;
  }
  *out = m;
  return GW_OK;
}

gw_status gw_mlp_destroy(gw_mlp* m) {
  if (!m) return GW_OK;
  (void)hipSetDevice(m->ctx->device);
  float* bufs[] = {m->p, m->g, m->m, m->v, m->ws};
  for (float* b : bufs)
    if (b) (void)hipFree(b);
  if (m->q) (void)hipFree(m->q);
  if (m->pre) (void)hipFree(m->pre);
  if (m->h_count) (void)hipHostFree(m->h_count);
  if (m->h_g) (void)hipHostFree(m->h_g);
  delete m;
  return GW_OK;
}

gw_status gw_mlp_n_params(int64_t* n) {
  if (!n) return set_error(GW_EINVAL, "gw_mlp_n_params: null");
  *n = kNPar;
  return GW_OK;
}

gw_status gw_mlp_set_scaling(gw_mlp* m, const double* x_mean, const double* x_std, double y_mean, double y_std) {
  if (!m || !x_mean || !x_std) return set_error(GW_EINVAL, "gw_mlp_set_scaling: null argument");
  for (int j = 0; j < kIn; ++j)
    if (!(x_std[j] > 0.0)) return set_error(GW_EINVAL, "gw_mlp_set_scaling: x_std must be > 0");
  if (!(y_std > 0.0) || !isfinite(y_mean)) return set_error(GW_EINVAL, "gw_mlp_set_scaling: bad y scaling");
  for (int j = 0; j < kIn; ++j) {
    m->sc.xm[j] = (float)x_mean[j];
    m->sc.xs_inv[j] = (float)(1.0 / x_std[j]);
  }
  m->sc.ym = y_mean;
  m->sc.ys = y_std;
  m->sc_version += 1;
  return GW_OK;
}

gw_status gw_mlp_set_params(gw_mlp* m, const float* host) {
  if (!m || !host) return set_error(GW_EINVAL, "gw_mlp_set_params: null argument");
  gw_status s = check_hip(hipMemcpy(m->p, host, kNPar * sizeof(float), hipMemcpyHostToDevice), "mlp copy");
  m->q_dirty = true;
  m->t = 0;
  if (s == GW_OK) s = check_hip(hipMemset(m->m, 0, kNPar * sizeof(float)), "mlp memset");
  if (s == GW_OK) s = check_hip(hipMemset(m->v, 0, kNPar * sizeof(float)), "mlp memset");
  return s;
}

gw_status gw_mlp_get_params(gw_mlp* m, float* host) {
  if (!m || !host) return set_error(GW_EINVAL, "gw_mlp_get_params: null argument");
  return check_hip(hipMemcpy(host, m->p, kNPar * sizeof(float), hipMemcpyDeviceToHost), "mlp copy");
}

gw_status gw_mlp_grad(gw_mlp* m, const double* x, const double* y, int64_t n, float* grads_host, float* loss_host,
                      void* stream) {
  if (!m || !x || !y || !grads_host) return set_error(GW_EINVAL, "gw_mlp_grad: null argument");
  if (n < 1 || n > (1 << 24)) return set_error(GW_EINVAL, "gw_mlp_grad: n out of range");
  hipStream_t st = (hipStream_t)stream;
  gw_status s = GW_OK;
  if (!m->h_g) s = check_hip(hipHostMalloc((void**)&m->h_g, (kNPar + 1) * sizeof(float)), "mlp pinned copy");
  if (s == GW_OK) s = grad32(m, x, y, n, st);
  // gradient and loss in one copy to pinned memory: two copies to pageable
  // memory took 20 us more of a call (1024 rows: 95 against 116)
  if (s == GW_OK)
    s = check_hip(hipMemcpyAsync(m->h_g, m->g, (kNPar + 1) * sizeof(float), hipMemcpyDeviceToHost, st), "copy");
  if (s == GW_OK) s = check_hip(hipStreamSynchronize(st), "gw_mlp_grad sync");
  if (s != GW_OK) return s;
  memcpy(grads_host, m->h_g, kNPar * sizeof(float));
  if (loss_host) *loss_host = m->h_g[kNPar];
  return s;
}

gw_status gw_mlp_train_step(gw_mlp* m, const double* x, const double* y, int64_t n, float lr, float* loss_host,
                            void* stream) {
  if (!m || !x || !y) return set_error(GW_EINVAL, "gw_mlp_train_step: null argument");
  if (n < 1 || n > (1 << 24)) return set_error(GW_EINVAL, "gw_mlp_train_step: n out of range");
  if (!(lr > 0.0f)) return set_error(GW_EINVAL, "gw_mlp_train_step: lr must be > 0");
  hipStream_t st = (hipStream_t)stream;
  gw_status s = grad32(m, x, y, n, st);
  if (s != GW_OK) return s;
  m->t += 1;
  const float c1 = (float)(1.0 / (1.0 - pow(0.9, (double)m->t)));
  const float c2 = (float)(1.0 / (1.0 - pow(0.999, (double)m->t)));
  hipLaunchKernelGGL(k_adam, dim3(nblk(kNPar)), dim3(256), 0, st, m->p, m->g, m->m, m->v, kNPar, lr, c1, c2);
  s = check_hip(hipGetLastError(), "adam launch");
  m->q_dirty = true;
  if (s == GW_OK && loss_host) {
    s = check_hip(hipMemcpyAsync(loss_host, m->loss, sizeof(float), hipMemcpyDeviceToHost, st), "copy");
    if (s == GW_OK) s = check_hip(hipStreamSynchronize(st), "gw_mlp_train_step sync");
  }
  return s;
}

gw_status gw_mlp_forward(gw_mlp* m, const double* x, int64_t n, double* out, int32_t use_bf16, void* stream) {
  if (!m || (n > 0 && (!x || !out))) return set_error(GW_EINVAL, "gw_mlp_forward: null argument");
  if (n < 0) return set_error(GW_EINVAL, "gw_mlp_forward: n < 0");
  if (n == 0) return GW_OK;
  hipStream_t st = (hipStream_t)stream;
  gw_status s = check_hip(hipSetDevice(m->ctx->device), "hipSetDevice");
  if (s != GW_OK) return s;
  if (use_bf16) {
    s = mlp_prepare(m, st);
    return s == GW_OK ? mlp_infer(m, x, n, out, st) : s;
  }
  const int64_t chunk = 1 << 16, most = std::min(n, chunk);
  s = mlp_ws(m, most * (1 + kIn + 2 * kH));
  for (int64_t o = 0; o < n && s == GW_OK; o += chunk) {
    const int64_t r = std::min(chunk, n - o);
    s = forward32(m, x + o * kIn, r, m->ws, m->ws + most, st);
    if (s == GW_OK) hipLaunchKernelGGL(k_unscale, dim3(nblk(r)), dim3(256), 0, st, m->ws, r, m->sc, out + o);
    if (s == GW_OK) s = check_hip(hipGetLastError(), "mlp forward");
  }
  return s;
}

// Prescreened exact evaluation of unit-cube candidates (see gwswig.h).
gw_status gw_prescreen_batch(gw_ctx* ctx, gw_mlp* m, const double* x, int64_t n, double logl_star, double margin,
                             double audit_frac, uint64_t seed, int32_t use_mlp, int32_t like, int32_t prec,
                             double* logl, double* pred, int32_t* flags, int64_t* n_exact, void* stream) {
  if (!ctx || !m || !n_exact) return set_error(GW_EINVAL, "gw_prescreen_batch: null argument");
  if (n < 0) return set_error(GW_EINVAL, "gw_prescreen_batch: n < 0");
  *n_exact = 0;
  if (n == 0) return GW_OK;
  if (!x || !logl || !flags) return set_error(GW_EINVAL, "gw_prescreen_batch: null pointer");
  if (!(audit_frac >= 0.0 && audit_frac <= 1.0) || !isfinite(margin))
    return set_error(GW_EINVAL, "gw_prescreen_batch: audit_frac in [0, 1] and finite margin");
  if (like != GW_FULL && like != GW_HET) return set_error(GW_EINVAL, "gw_prescreen_batch: bad like");
  if (like == GW_HET && !ctx->het) return set_error(GW_ESTATE, "gw_prescreen_batch: heterodyne_setup missing");
  if (ctx->n_dist <= 0) return set_error(GW_ESTATE, "gw_prescreen_batch: distance marginal needs a distance grid");
  hipStream_t st = (hipStream_t)stream;
  gw_status s = check_hip(hipSetDevice(ctx->device), "hipSetDevice");
  if (s != GW_OK) return s;
  // workspace: pred [n], pos [n + 1], x_sel [n][11], theta [n][13], logl_sel [n]
  const int64_t need = n * (1 + 1 + kIn + 13 + 1) + 1;
  if (!m->h_count) {
    s = check_hip(hipHostMalloc((void**)&m->h_count, sizeof(int64_t), hipHostMallocDefault), "pinned count");
    if (s != GW_OK) return s;
  }
  if (m->pre_cap < need) {
    if (m->pre) (void)hipFree(m->pre);
    m->pre = nullptr;
    m->pre_cap = 0;
    s = check_hip(hipMalloc(&m->pre, need * sizeof(double)), "prescreen workspace");
    if (s != GW_OK) return s;
    m->pre_cap = need;
  }
  double* d_pred = (double*)m->pre;
  int64_t* d_pos = (int64_t*)(d_pred + n);
  double* d_xs = (double*)(d_pos + n + 1);
  double* d_th = d_xs + n * kIn;
  double* d_sub = d_th + n * 13;
  if (use_mlp) {
    s = gw_mlp_forward(m, x, n, d_pred, 1, st);
    if (s != GW_OK) return s;
  }
  hipLaunchKernelGGL(k_prescreen_flags, dim3(nblk(n)), dim3(256), 0, st, (const double*)d_pred, n,
                     logl_star - margin, audit_frac, seed, use_mlp, flags);
  hipLaunchKernelGGL(k_select_scan, dim3(1), dim3(256), 0, st, (const int32_t*)flags, n, d_pos);
  hipLaunchKernelGGL(k_gather_rows, dim3(nblk(n)), dim3(256), 0, st, x, n, (const int32_t*)flags,
                     (const int64_t*)d_pos, d_xs);
  s = check_hip(hipGetLastError(), "prescreen launch");
  if (s == GW_OK)
    s = check_hip(hipMemcpyAsync(m->h_count, d_pos + n, sizeof(int64_t), hipMemcpyDeviceToHost, st), "copy");
  if (s == GW_OK) s = check_hip(hipStreamSynchronize(st), "prescreen count");
  if (s != GW_OK) return s;
  const int64_t ns = *m->h_count;
  if (ns > 0) {
    s = gw_prior_transform(ctx, d_xs, ns, d_th, stream);
    if (s == GW_OK) s = loglike_batch(ctx, d_th, ns, like, GW_MARG_PHASE_DIST, prec, d_sub, stream);
    if (s != GW_OK) return s;
  }
  hipLaunchKernelGGL(k_scatter_logl, dim3(nblk(n)), dim3(256), 0, st, (const double*)d_sub, n, (const int32_t*)flags,
                     (const int64_t*)d_pos, logl);
  s = check_hip(hipGetLastError(), "prescreen scatter launch");
  if (s == GW_OK && pred && use_mlp)
    s = check_hip(hipMemcpyAsync(pred, d_pred, n * sizeof(double), hipMemcpyDeviceToDevice, st), "copy");
  *n_exact = ns;
  return s;
}

}  // extern "C"
