// The optimiser's update as a device kernel, for parameters whose optimiser state lives in HBM
// (karma_config.device_update_first): the tensors of the first record are the last the backward
// pass completes and the first the next forward pass reads, so a host update of them (gradient
// copy out, update, weight copy back) cannot hide behind anything; updated where they are, the
// step has no such tail.  Same arithmetic as the host loops (csrc/host_optim_loops.h): fp32
// master weights and moments, bias-corrected Adam without weight decay, SGD with momentum
// without dampening, plain SGD; the device copy of the weight is rounded to nearest even.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "device_utils.h"
#include "karma.h"
#include "kernels.h"

namespace karma {
namespace {

// The tensors of one launch: block b works on the tensor whose blocks [first[t], first[t + 1]) it is among.
struct UpdateSet {
  OptimTensor t[OPTIM_TENSORS];
  unsigned first[OPTIM_TENSORS + 1];
  int n;
};

template <int KIND, bool G_BF16, bool O_BF16>
__device__ __forceinline__ void update_tensor(const OptimTensor& p, size_t i, size_t stride, float lr, float beta1, float beta2, float eps,
                                              float c1, float c2) {
  float* __restrict__ w = p.w;
  float* __restrict__ m = p.m;
  float* __restrict__ v = p.v;
  const void* __restrict__ g = p.g;
  void* __restrict__ out = p.out;
  for (; i < p.n; i += stride) {
    const float gi = G_BF16 ? bf2f(((const bf16_t*)g)[i]) : ((const float*)g)[i];
    float nw;
    if (KIND == KARMA_OPT_ADAM) {
      const float mi = beta1 * m[i] + (1.0f - beta1) * gi;
      const float vi = beta2 * v[i] + (1.0f - beta2) * gi * gi;
      m[i] = mi;
      v[i] = vi;
      nw = w[i] - lr * (mi * c1) / (sqrtf(vi * c2) + eps);
    } else if (KIND == KARMA_OPT_SGD_MOMENTUM) {
      const float bi = beta1 * m[i] + gi;
      m[i] = bi;
      nw = w[i] - lr * bi;
    } else {
      nw = w[i] - lr * gi;
    }
    w[i] = nw;
    if (O_BF16) ((bf16_t*)out)[i] = f2bf(nw);
    else ((float*)out)[i] = nw;
  }
}

// All tensors of a record in one launch: most are vectors of a few hundred values, and a launch each cost 4.7 us.
template <int KIND>
__global__ __launch_bounds__(256) void optim_update_kernel(UpdateSet u, float lr, float beta1, float beta2, float eps, float c1, float c2) {
  int k = 0;
  while (k + 1 < u.n && blockIdx.x >= u.first[k + 1]) ++k;
  const OptimTensor p = u.t[k];
  const unsigned block = blockIdx.x - u.first[k], blocks = u.first[k + 1] - u.first[k];
  const size_t i = (size_t)block * 256 + threadIdx.x, stride = (size_t)blocks * 256;
  if (p.g_bf16 && p.out_bf16) update_tensor<KIND, true, true>(p, i, stride, lr, beta1, beta2, eps, c1, c2);
  else if (p.g_bf16) update_tensor<KIND, true, false>(p, i, stride, lr, beta1, beta2, eps, c1, c2);
  else if (p.out_bf16) update_tensor<KIND, false, true>(p, i, stride, lr, beta1, beta2, eps, c1, c2);
  else update_tensor<KIND, false, false>(p, i, stride, lr, beta1, beta2, eps, c1, c2);
}

}  // namespace

int optim_update_dev(int kind, const OptimTensor* tensors, int n, float lr, float beta1, float beta2, float eps, uint64_t step, hipStream_t s) {
  if (!tensors || n <= 0 || n > OPTIM_TENSORS) return KARMA_E_INVAL;
  const float c1 = (float)(1.0 / (1.0 - std::pow((double)beta1, (double)step)));
  const float c2 = (float)(1.0 / (1.0 - std::pow((double)beta2, (double)step)));
  UpdateSet u{};
  u.n = n;
  for (int k = 0; k < n; ++k) {
    const OptimTensor& t = tensors[k];
    if (!t.w || !t.g || !t.out || !t.n) return KARMA_E_INVAL;
    if ((kind == KARMA_OPT_ADAM && (!t.m || !t.v)) || (kind == KARMA_OPT_SGD_MOMENTUM && !t.m)) return KARMA_E_INVAL;
    u.t[k] = t;
    u.first[k + 1] = u.first[k] + (unsigned)std::min<size_t>((t.n + 255) / 256, 256 * 16);
  }
#define KARMA_OPT_LAUNCH(K) hipLaunchKernelGGL(optim_update_kernel<K>, dim3(u.first[n]), dim3(256), 0, s, u, lr, beta1, beta2, eps, c1, c2)
  if (kind == KARMA_OPT_ADAM) KARMA_OPT_LAUNCH(KARMA_OPT_ADAM);
  else if (kind == KARMA_OPT_SGD_MOMENTUM) KARMA_OPT_LAUNCH(KARMA_OPT_SGD_MOMENTUM);
  else if (kind == KARMA_OPT_SGD) KARMA_OPT_LAUNCH(KARMA_OPT_SGD);
  else return KARMA_E_INVAL;
#undef KARMA_OPT_LAUNCH
  return hipGetLastError() == hipSuccess ? KARMA_OK : KARMA_E_HIP;
}

}  // namespace karma
