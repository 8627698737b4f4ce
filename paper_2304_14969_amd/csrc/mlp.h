// Separability-proposal network (internal).
#pragma once

#include <hip/hip_runtime.h>

#include "../../include/qs.h"

struct qs_mlp {
  void* block = nullptr;  // P, M, V, G (parameters, Adam moments, gradient)
  float* P = nullptr;
  float* M = nullptr;
  float* V = nullptr;
  float* G = nullptr;
  hipStream_t stream = nullptr;
  float* hscore = nullptr;  // pinned, mapped: kScoreRows x 32 inputs, then kScoreRows logits
  float* dscore = nullptr;  // its device address
};

namespace qs {
constexpr int kScoreRows = 64;  // rows scored through the pinned staging
int mlp_param_count();
// One wavefront per row; X and logit may be mapped host memory.
hipError_t launch_mlp_score(const float* P, const float* X, int rows, float* logit,
                            hipStream_t s);
// The many-row kernels run at most kMlpGroups workgroups; mlp_groups(rows) is
// their number for `rows` rows, the length of `loss` (the workgroups' sums of
// the rows' cross-entropies) and, times mlp_param_count(), of `part` (their
// partial gradients).
constexpr int kMlpGroups = 256;
int mlp_groups(int rows);
// scores[r] = sigmoid(logit of row r)
hipError_t launch_mlp_scores(const float* P, const float* X, int rows, float* scores,
                             hipStream_t s);
hipError_t launch_mlp_loss(const float* P, const float* X, const float* y, int rows, double* loss,
                           hipStream_t s);
// Gradient G of the mean cross-entropy of the rows.
hipError_t launch_mlp_grad(const float* P, const float* X, const float* y, int rows, float* part,
                           double* loss, float* G, hipStream_t s);
// One Adam step on the rows (c1, c2: the bias corrections 1 / (1 - beta^t)).
hipError_t launch_mlp_step(float* P, float* M, float* V, const float* X, const float* y, int rows,
                           float* part, double* loss, float lr, float b1, float b2, float eps,
                           float c1, float c2, hipStream_t s);
// sigmoid scores of host rows (rows x 32) on the network's stream; synchronizes
int mlp_scores(qs_mlp* net, const float* X, uint64_t rows, float* scores);
}  // namespace qs
