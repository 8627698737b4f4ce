// Separability-proposal network on the GPU: 32 -> 64 (tanh) -> 64 (tanh) -> 1
// logit; score = sigmoid(logit). Float32 forward, backward and Adam.
//
// Parameter vector (6,337 floats): W1[32][64], b1[64], W2[64][64], b2[64],
// W3[64], b3 -- row-major, x @ W + b.
#include "mlp.h"

namespace qs {
namespace {

constexpr int kIn = 32, kH = 64;
constexpr int oW1 = 0, oB1 = oW1 + kIn * kH, oW2 = oB1 + kH, oB2 = oW2 + kH * kH, oW3 = oB2 + kH,
              oB3 = oW3 + kH, kParams = oB3 + 1;
constexpr int kBlock = 256;

// Forward pass, loss and gradient of many rows. A workgroup of 4 wavefronts
// takes 16 rows at a time; wavefront w owns hidden units 16 w .. 16 w + 15 of
// both layers, its columns of the weights (40 values a lane) stay in
// registers, and every product is 16 x 16 x 4 FP32 matrix-core steps: lane (q,
// col) = (lane / 16, lane % 16) supplies A[row = col][k = q] and B[k = q][unit =
// col] and holds rows 4 q + i of unit col in its 4 result registers, so the
// activations a lane computed are the ones it needs again for tanh'. Between
// the layers the 16 x 64 activations pass through LDS.
//
// The gradient X^T D1, H1^T D2 is the same kind of product with the rows as
// the inner dimension; each workgroup keeps its 24 tiles in registers over all
// the rows it takes and writes one partial gradient, and k_mlp_reduce adds the
// partials in workgroup order (in float64). Its bound is latency: 16 rows pass
// seven barriers and 64 matrix steps in each wavefront, and a minibatch of 256 rows is 16
// workgroups (10.4 us, then 3.2 us for the sums and the Adam step). 40 steps
// of 256 rows, then loss, gradient and scores of 20000 rows take 1.07 ms
// (0.6 ms of it on the GPU, the rest copies of the rows) instead of 18.7 ms
// with one thread per row (forward 58 us, deltas 45 us a launch) and one
// thread per weight that walked all the rows (319 us a launch); the gradient's
// error against float64 fell from 2.0e-6 to 5e-7.
enum MlpMode { kScores, kLoss, kGrad };
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kRows = 16;          // rows a workgroup takes at a time
constexpr int kPadX = kIn + 1, kPadH = kH + 1;

template <MlpMode MODE>
__global__ void __launch_bounds__(kBlock) k_mlp_rows(const float* __restrict__ P,
                                                     const float* __restrict__ X,
                                                     const float* __restrict__ y, int rows,
                                                     float* __restrict__ scores,
                                                     float* __restrict__ part,
                                                     double* __restrict__ loss) {
  __shared__ float sx[kRows * kPadX], s2[kRows * kPadH], sz[4 * kRows];
  __shared__ __align__(16) float s1[kRows * kPadH];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, q = lane >> 4, col = lane & 15;
  const int j = 16 * w + col;  // this lane's hidden unit
  float w1[kIn / 4], w2[kH / 4], w2t[kH / 4];
#pragma unroll
  for (int s = 0; s < kIn / 4; ++s) w1[s] = P[oW1 + (4 * s + q) * kH + j];
#pragma unroll
  for (int s = 0; s < kH / 4; ++s) w2[s] = P[oW2 + (4 * s + q) * kH + j];
  if constexpr (MODE == kGrad) {
#pragma unroll
    for (int s = 0; s < kH / 4; ++s) w2t[s] = P[oW2 + j * kH + 4 * s + q];
  }
  const float b1 = P[oB1 + j], b2 = P[oB2 + j], w3 = P[oW3 + j], b3 = P[oB3];
  f32x4 g1[kIn / 16] = {}, g2[kH / 16] = {};
  float gb1 = 0, gb2 = 0, gw3 = 0, gb3 = 0;
  double ls = 0;
  const int nblk = (rows + kRows - 1) / kRows;
  for (int blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
    // Rows past the end are zeros in every array, as products by a zero factor
    // alone are NaN where a weight has grown infinite.
    const int r0 = blk * kRows, left = rows - r0;
#pragma unroll
    for (int e = threadIdx.x; e < kRows * kIn; e += kBlock) {
      const int r = e / kIn;
      sx[r * kPadX + e % kIn] = r < left ? X[size_t(r0) * kIn + e] : 0.0f;
    }
    __syncthreads();
    f32x4 h1 = {b1, b1, b1, b1};
#pragma unroll
    for (int s = 0; s < kIn / 4; ++s)
      h1 = __builtin_amdgcn_mfma_f32_16x16x4f32(sx[col * kPadX + 4 * s + q], w1[s], h1, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      h1[i] = tanhf(h1[i]);
      if (left < kRows && 4 * q + i >= left) h1[i] = 0.0f;
      s1[(4 * q + i) * kPadH + j] = h1[i];
    }
    __syncthreads();
    f32x4 h2 = {b2, b2, b2, b2};
#pragma unroll
    for (int s = 0; s < kH / 4; ++s)
      h2 = __builtin_amdgcn_mfma_f32_16x16x4f32(s1[col * kPadH + 4 * s + q], w2[s], h2, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      h2[i] = tanhf(h2[i]);
      if (left < kRows && 4 * q + i >= left) h2[i] = 0.0f;
      float v = h2[i] * w3;  // summed over the wavefront's 16 units
#pragma unroll
      for (int off = 8; off > 0; off >>= 1) v += __shfl_xor(v, off, 16);
      if (col == 0) sz[w * kRows + 4 * q + i] = v;
    }
    __syncthreads();
    auto logit = [&](int r) {
      return b3 + ((sz[r] + sz[kRows + r]) + (sz[2 * kRows + r] + sz[3 * kRows + r]));
    };
    if (threadIdx.x < kRows && int(threadIdx.x) < left) {
      const int r = threadIdx.x;
      const float z = logit(r);
      if constexpr (MODE == kScores) {
        scores[r0 + r] = 1.0f / (1.0f + expf(-z));
      } else {
        ls += double(fmaxf(z, 0.0f) - y[r0 + r] * z + log1pf(expf(-fabsf(z))));
      }
    }
    if constexpr (MODE == kGrad) {
      // mean binary cross-entropy: dz3 = (sigmoid(z) - y) / rows,
      // dz2 = dz3 W3 (1 - h2^2), dz1 = (dz2 W2^T) (1 - h1^2)
      float d3[4], d2[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = 4 * q + i;
        const float yr = r < left ? y[r0 + r] : 0.0f;
        d3[i] = r < left ? (1.0f / (1.0f + expf(-logit(r))) - yr) / float(rows) : 0.0f;
        d2[i] = d3[i] * w3 * (1.0f - h2[i] * h2[i]);
        if (left < kRows && r >= left) d2[i] = 0.0f;
        s2[r * kPadH + j] = d2[i];
        gw3 += h2[i] * d3[i];
        gb2 += d2[i];
        gb3 += d3[i];
      }
      __syncthreads();
      f32x4 d1 = {};
#pragma unroll
      for (int s = 0; s < kH / 4; ++s)
        d1 = __builtin_amdgcn_mfma_f32_16x16x4f32(s2[col * kPadH + 4 * s + q], w2t[s], d1, 0, 0, 0);
      // weights of layer 2: rows r = 4 s + q of H1 (16 units at 16 a) and D2
#pragma unroll
      for (int s = 0; s < kRows / 4; ++s) {
        const float b = s2[(4 * s + q) * kPadH + j];
#pragma unroll
        for (int a = 0; a < kH / 16; ++a)
          g2[a] = __builtin_amdgcn_mfma_f32_16x16x4f32(s1[(4 * s + q) * kPadH + 16 * a + col], b,
                                                       g2[a], 0, 0, 0);
      }
      __syncthreads();  // D2 is read; its place takes D1
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        d1[i] *= 1.0f - h1[i] * h1[i];
        if (left < kRows && 4 * q + i >= left) d1[i] = 0.0f;
        s2[(4 * q + i) * kPadH + j] = d1[i];
        gb1 += d1[i];
      }
      __syncthreads();
#pragma unroll
      for (int s = 0; s < kRows / 4; ++s) {
        const float b = s2[(4 * s + q) * kPadH + j];
#pragma unroll
        for (int a = 0; a < kIn / 16; ++a)
          g1[a] = __builtin_amdgcn_mfma_f32_16x16x4f32(sx[(4 * s + q) * kPadX + 16 * a + col], b,
                                                       g1[a], 0, 0, 0);
      }
    }
    __syncthreads();
  }
  if constexpr (MODE != kScores) {
    // the 16 row sums of the loss, in row order
    double* sd = reinterpret_cast<double*>(s1);
    if (threadIdx.x < kRows) sd[threadIdx.x] = ls;
    __syncthreads();
    if (threadIdx.x == 0) {
      double t = 0;
      for (int r = 0; r < kRows; ++r) t += sd[r];
      loss[blockIdx.x] = t;
    }
  }
  if constexpr (MODE == kGrad) {
    float* g = part + size_t(blockIdx.x) * kParams;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
      for (int a = 0; a < kIn / 16; ++a) g[oW1 + (16 * a + 4 * q + i) * kH + j] = g1[a][i];
#pragma unroll
      for (int a = 0; a < kH / 16; ++a) g[oW2 + (16 * a + 4 * q + i) * kH + j] = g2[a][i];
    }
    // column sums over the four row groups of the wavefront
    auto over_q = [](float v) {
      v += __shfl_xor(v, 16, 64);
      return v + __shfl_xor(v, 32, 64);
    };
    gb1 = over_q(gb1);
    gb2 = over_q(gb2);
    gw3 = over_q(gw3);
    gb3 = over_q(gb3);
    if (q == 0) {
      g[oB1 + j] = gb1;
      g[oB2 + j] = gb2;
      g[oW3 + j] = gw3;
      if (j == 0) g[oB3] = gb3;
    }
  }
}

// Adds the workgroups' partial gradients in order (float64), then either
// stores the gradient or takes one Adam step with it (bias-corrected moments;
// c1 = 1/(1-beta1^t), c2 = 1/(1-beta2^t)).
struct AdamStep {
  float lr, b1, b2, eps, c1, c2;
};

template <bool ADAM>
__global__ void __launch_bounds__(kH) k_mlp_reduce(const float* __restrict__ part, int parts,
                                                   float* __restrict__ G, float* __restrict__ P,
                                                   float* __restrict__ M, float* __restrict__ V,
                                                   AdamStep st) {
  const int p = blockIdx.x * kH + threadIdx.x;
  if (p >= kParams) return;
  double t = 0;
#pragma unroll 16
  for (int k = 0; k < parts; ++k) t += part[size_t(k) * kParams + p];
  const float g = float(t);
  if constexpr (ADAM) {
    const float m = st.b1 * M[p] + (1.0f - st.b1) * g;
    const float v = st.b2 * V[p] + (1.0f - st.b2) * g * g;
    M[p] = m;
    V[p] = v;
    P[p] -= st.lr * (m * st.c1) / (sqrtf(v * st.c2) + st.eps);
  } else {
    G[p] = g;
  }
}

// Scoring of a few rows: one wavefront per row, lane j owns hidden unit j of
// both layers (weight columns read coalesced), the output dot product summed
// across the wavefront in a fixed butterfly order. X and logit may live in
// mapped host memory.
__global__ void __launch_bounds__(kH) k_mlp_score(const float* __restrict__ P,
                                                  const float* __restrict__ X,
                                                  float* __restrict__ logit) {
  __shared__ float x[kIn], h1[kH];
  const int r = blockIdx.x, j = threadIdx.x;
  if (j < kIn) x[j] = X[size_t(r) * kIn + j];
  __syncthreads();
  float s = P[oB1 + j];
#pragma unroll 8
  for (int i = 0; i < kIn; ++i) s += x[i] * P[oW1 + i * kH + j];
  h1[j] = tanhf(s);
  __syncthreads();
  float s2 = P[oB2 + j];
#pragma unroll 8
  for (int i = 0; i < kH; ++i) s2 += h1[i] * P[oW2 + i * kH + j];
  float v = tanhf(s2) * P[oW3 + j];
#pragma unroll
  for (int off = kH / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kH);
  if (j == 0) logit[r] = v + P[oB3];
}

unsigned row_groups(int rows) {
  const int blks = (rows + kRows - 1) / kRows;
  return unsigned(blks < kMlpGroups ? blks : kMlpGroups);
}

}  // namespace

int mlp_param_count() { return kParams; }
int mlp_groups(int rows) { return int(row_groups(rows)); }

hipError_t launch_mlp_score(const float* P, const float* X, int rows, float* logit,
                            hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_score, dim3(rows), dim3(kH), 0, s, P, X, logit);
  return hipGetLastError();
}

hipError_t launch_mlp_scores(const float* P, const float* X, int rows, float* scores,
                             hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_mlp_rows<kScores>, dim3(row_groups(rows)), dim3(kBlock), 0, s, P, X,
                     nullptr, rows, scores, nullptr, nullptr);
  return hipGetLastError();
}

hipError_t launch_mlp_loss(const float* P, const float* X, const float* y, int rows, double* loss,
                           hipStream_t s) {
  if (rows <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_mlp_rows<kLoss>, dim3(row_groups(rows)), dim3(kBlock), 0, s, P, X, y, rows,
                     nullptr, nullptr, loss);
  return hipGetLastError();
}

hipError_t launch_mlp_grad(const float* P, const float* X, const float* y, int rows, float* part,
                           double* loss, float* G, hipStream_t s) {
  if (rows <= 0) return hipErrorInvalidValue;
  const unsigned groups = row_groups(rows);
  hipLaunchKernelGGL(k_mlp_rows<kGrad>, dim3(groups), dim3(kBlock), 0, s, P, X, y, rows, nullptr,
                     part, loss);
  hipLaunchKernelGGL(k_mlp_reduce<false>, dim3((kParams + kH - 1) / kH), dim3(kH), 0, s, part,
                     int(groups), G, nullptr, nullptr, nullptr, AdamStep{});
  return hipGetLastError();
}

hipError_t launch_mlp_step(float* P, float* M, float* V, const float* X, const float* y, int rows,
                           float* part, double* loss, float lr, float b1, float b2, float eps,
                           float c1, float c2, hipStream_t s) {
  if (rows <= 0) return hipErrorInvalidValue;
  const unsigned groups = row_groups(rows);
  hipLaunchKernelGGL(k_mlp_rows<kGrad>, dim3(groups), dim3(kBlock), 0, s, P, X, y, rows, nullptr,
                     part, loss);
  hipLaunchKernelGGL(k_mlp_reduce<true>, dim3((kParams + kH - 1) / kH), dim3(kH), 0, s, part,
                     int(groups), nullptr, P, M, V, AdamStep{lr, b1, b2, eps, c1, c2});
  return hipGetLastError();
}

}  // namespace qs
