// Host side of the separability-proposal network: parameter storage on the
// device, forward passes for scoring, gradients and Adam training, all run by
// the kernels of k_mlp.hip.
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <vector>

#include "mlp.h"
#include "qs_internal.h"

namespace qs {
void* device_alloc(size_t bytes);
void device_free(void* p);
void set_last_error(const char* msg);
}  // namespace qs

namespace {

constexpr int kScoreRowsFloats = qs::kScoreRows * (QS_MLP_INPUTS + 1);

int mfail(int code, const char* fmt, ...) {
  char buf[256];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  qs::set_last_error(buf);
  return code;
}

int merr(hipError_t e, const char* what) {
  if (e == hipSuccess) return QS_OK;
  return mfail(QS_E_DEVICE, "%s: %s", what, hipGetErrorString(e));
}

// Device scratch: X and, with labels, y of `rows` rows; `parts` partial
// gradients and losses of the workgroups; scores.
struct Scratch {
  float *X = nullptr, *y = nullptr, *part = nullptr, *scores = nullptr;
  double* loss = nullptr;
  void* block = nullptr;
  bool alloc(uint64_t rows, bool labels, uint64_t parts, bool grads, bool want_scores) {
    const size_t np = size_t(qs::mlp_param_count());
    const size_t f = rows * QS_MLP_INPUTS + (labels ? rows : 0) + (want_scores ? rows : 0) +
                     (grads ? parts * np : 0);
    block = qs::device_alloc(parts * sizeof(double) + f * sizeof(float));
    if (!block) return false;
    loss = static_cast<double*>(block);
    float* p = reinterpret_cast<float*>(loss + parts);
    X = p; p += rows * QS_MLP_INPUTS;
    if (labels) { y = p; p += rows; }
    if (want_scores) { scores = p; p += rows; }
    if (grads) part = p;
    return true;
  }
  ~Scratch() { qs::device_free(block); }
};

// The mean of the rows' losses from the workgroups' sums (in order).
double mean_loss(const double* sums, int n, uint64_t rows) {
  double t = 0.0;
  for (int i = 0; i < n; ++i) t += sums[i];
  return t / double(rows);
}

}  // namespace

namespace qs {

// scores[r] = sigmoid(logit) of the rows of host X (rows x 32); synchronizes.
int mlp_scores(qs_mlp* net, const float* X, uint64_t rows, float* scores) {
  if (rows == 0) return QS_OK;
  if (rows <= uint64_t(kScoreRows)) {
    // the usual case (the dirty qubits of one separation round): the kernel
    // reads the rows from and writes the logits to mapped pinned memory
    float* hz = net->hscore + kScoreRows * QS_MLP_INPUTS;
    float* dz = net->dscore + kScoreRows * QS_MLP_INPUTS;
    std::memcpy(net->hscore, X, rows * QS_MLP_INPUTS * sizeof(float));
    hipError_t e = launch_mlp_score(net->P, net->dscore, int(rows), dz, net->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(net->stream);
    if (int rc = merr(e, "network forward")) return rc;
    for (uint64_t r = 0; r < rows; ++r) scores[r] = 1.0f / (1.0f + std::exp(-hz[r]));
    return QS_OK;
  }
  Scratch s;
  if (!s.alloc(rows, false, 0, false, true)) return mfail(QS_E_NOMEM, "network scratch");
  hipError_t e = hipMemcpyAsync(s.X, X, rows * QS_MLP_INPUTS * sizeof(float), hipMemcpyHostToDevice,
                                net->stream);
  if (e == hipSuccess) e = launch_mlp_scores(net->P, s.X, int(rows), s.scores, net->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(scores, s.scores, rows * sizeof(float), hipMemcpyDeviceToHost, net->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(net->stream);
  return merr(e, "network forward");
}

}  // namespace qs

extern "C" {

int qs_mlp_create(qs_mlp** out) {
  if (!out) return mfail(QS_E_INVAL, "out is NULL");
  qs_mlp* n = new qs_mlp();
  const int np = qs::mlp_param_count();
  void* blk = qs::device_alloc(size_t(4) * np * sizeof(float));
  if (!blk) {
    delete n;
    return mfail(QS_E_NOMEM, "network parameters");
  }
  const size_t score_floats = size_t(kScoreRowsFloats);
  if (hipHostMalloc(reinterpret_cast<void**>(&n->hscore), score_floats * sizeof(float),
                    hipHostMallocMapped) != hipSuccess ||
      hipHostGetDevicePointer(reinterpret_cast<void**>(&n->dscore), n->hscore, 0) != hipSuccess) {
    if (n->hscore) (void)hipHostFree(n->hscore);
    qs::device_free(blk);
    delete n;
    return mfail(QS_E_NOMEM, "network scoring buffers");
  }
  n->block = blk;
  n->P = static_cast<float*>(blk);
  n->M = n->P + np;
  n->V = n->M + np;
  n->G = n->V + np;
  std::vector<float> zero(size_t(4) * np, 0.0f);
  hipError_t e = hipMemcpy(blk, zero.data(), zero.size() * sizeof(float), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    (void)hipHostFree(n->hscore);
    qs::device_free(blk);
    delete n;
    return merr(e, "network init");
  }
  *out = n;
  return QS_OK;
}

int qs_mlp_free(qs_mlp* n) {
  if (!n) return QS_OK;
  (void)hipStreamSynchronize(n->stream);
  qs::device_free(n->block);
  (void)hipHostFree(n->hscore);
  delete n;
  return QS_OK;
}

int qs_mlp_set_stream(qs_mlp* n, void* stream) {
  if (!n) return mfail(QS_E_INVAL, "network is NULL");
  n->stream = static_cast<hipStream_t>(stream);
  return QS_OK;
}

int qs_mlp_set_params(qs_mlp* n, const float* host, uint64_t count) {
  if (!n || !host) return mfail(QS_E_INVAL, "NULL argument");
  if (count != uint64_t(QS_MLP_PARAMS)) return mfail(QS_E_INVAL, "expected %d parameters", QS_MLP_PARAMS);
  for (uint64_t i = 0; i < count; ++i)
    if (!std::isfinite(host[i])) return mfail(QS_E_INVAL, "parameter %llu is not finite", (unsigned long long)i);
  hipError_t e = hipMemcpyAsync(n->P, host, count * sizeof(float), hipMemcpyHostToDevice, n->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(n->stream);
  return merr(e, "set params");
}

int qs_mlp_get_params(qs_mlp* n, float* host, uint64_t count) {
  if (!n || !host) return mfail(QS_E_INVAL, "NULL argument");
  if (count != uint64_t(QS_MLP_PARAMS)) return mfail(QS_E_INVAL, "expected %d parameters", QS_MLP_PARAMS);
  hipError_t e = hipMemcpyAsync(host, n->P, count * sizeof(float), hipMemcpyDeviceToHost, n->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(n->stream);
  return merr(e, "get params");
}

int qs_mlp_forward(qs_mlp* n, const float* X, uint64_t rows, float* scores) {
  if (!n || (rows && (!X || !scores))) return mfail(QS_E_INVAL, "NULL argument");
  if (rows > (uint64_t(1) << 30)) return mfail(QS_E_INVAL, "too many rows");
  return qs::mlp_scores(n, X, rows, scores);
}

int qs_mlp_grad(qs_mlp* n, const float* X, const float* y, uint64_t rows, float* grad,
                double* loss) {
  if (!n || !X || !y || !grad) return mfail(QS_E_INVAL, "NULL argument");
  if (rows == 0 || rows > (uint64_t(1) << 24)) return mfail(QS_E_INVAL, "rows = %llu", (unsigned long long)rows);
  Scratch s;
  const int groups = qs::mlp_groups(int(rows));
  if (!s.alloc(rows, true, groups, true, false)) return mfail(QS_E_NOMEM, "network scratch");
  hipError_t e = hipMemcpyAsync(s.X, X, rows * QS_MLP_INPUTS * sizeof(float), hipMemcpyHostToDevice, n->stream);
  if (e == hipSuccess) e = hipMemcpyAsync(s.y, y, rows * sizeof(float), hipMemcpyHostToDevice, n->stream);
  if (e == hipSuccess)
    e = qs::launch_mlp_grad(n->P, s.X, s.y, int(rows), s.part, s.loss, n->G, n->stream);
  double sums[qs::kMlpGroups];
  if (e == hipSuccess)
    e = hipMemcpyAsync(grad, n->G, QS_MLP_PARAMS * sizeof(float), hipMemcpyDeviceToHost, n->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(sums, s.loss, groups * sizeof(double), hipMemcpyDeviceToHost, n->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(n->stream);
  if (int rc = merr(e, "network gradient")) return rc;
  if (loss) *loss = mean_loss(sums, groups, rows);
  return QS_OK;
}

int qs_mlp_train(qs_mlp* n, const float* X, const float* y, uint64_t rows, const qs_train_cfg* cfg,
                 double* final_loss) {
  if (!n || !X || !y || !cfg) return mfail(QS_E_INVAL, "NULL argument");
  if (rows == 0 || rows > (uint64_t(1) << 26)) return mfail(QS_E_INVAL, "rows = %llu", (unsigned long long)rows);
  const uint64_t B = cfg->batch ? cfg->batch : 256;
  if (B > rows) return mfail(QS_E_INVAL, "batch larger than the data");
  if (!(cfg->lr > 0) || !(cfg->beta1 >= 0 && cfg->beta1 < 1) || !(cfg->beta2 >= 0 && cfg->beta2 < 1))
    return mfail(QS_E_INVAL, "bad optimizer settings");
  // the whole data set on the device, minibatches are consecutive rows
  Scratch data;
  const int groups = qs::mlp_groups(int(rows));  // at least those of a minibatch
  if (!data.alloc(rows, true, groups, true, false)) return mfail(QS_E_NOMEM, "training buffers");
  hipError_t e = hipMemcpyAsync(data.X, X, rows * QS_MLP_INPUTS * sizeof(float), hipMemcpyHostToDevice, n->stream);
  if (e == hipSuccess) e = hipMemcpyAsync(data.y, y, rows * sizeof(float), hipMemcpyHostToDevice, n->stream);
  // fresh optimizer moments
  if (e == hipSuccess)
    e = hipMemsetAsync(n->M, 0, size_t(2) * QS_MLP_PARAMS * sizeof(float), n->stream);
  double b1t = 1.0, b2t = 1.0;
  uint64_t cursor = 0;
  for (uint32_t step = 1; step <= cfg->steps && e == hipSuccess; ++step) {
    if (cursor + B > rows) cursor = 0;
    const float* Xb = data.X + cursor * QS_MLP_INPUTS;
    const float* yb = data.y + cursor;
    cursor += B;
    b1t *= cfg->beta1;
    b2t *= cfg->beta2;
    e = qs::launch_mlp_step(n->P, n->M, n->V, Xb, yb, int(B), data.part, data.loss, cfg->lr,
                            cfg->beta1, cfg->beta2, cfg->eps, float(1.0 / (1.0 - b1t)),
                            float(1.0 / (1.0 - b2t)), n->stream);
  }
  if (e == hipSuccess && final_loss) {
    // mean loss over the whole data set with the trained parameters
    double sums[qs::kMlpGroups];
    e = qs::launch_mlp_loss(n->P, data.X, data.y, int(rows), data.loss, n->stream);
    if (e == hipSuccess)
      e = hipMemcpyAsync(sums, data.loss, groups * sizeof(double), hipMemcpyDeviceToHost, n->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(n->stream);
    if (e == hipSuccess) *final_loss = mean_loss(sums, groups, rows);
  }
  if (e == hipSuccess) e = hipStreamSynchronize(n->stream);
  return merr(e, "network training");
}

}  // extern "C"
