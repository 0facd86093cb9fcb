// Parameter-side kernels: the packed weight copies the MFMA kernels read
// (FP32 or round-to-nearest-even BF16, in 16-byte lane-fragment order) and the
// Adam update of the flat FP32 parameters.
#include <algorithm>
#include <cmath>

#include "device_common.h"
#include "fvan_internal.h"

namespace fvan {

// One packed matrix: dst = pack of the [rows x K] matrix M, M[r][k] = src[r*K + k]
// (or src[k*rows + r] when transposed, i.e. M = W^T of a row-major W [K x rows]).
// Split mode writes the bf16 hi parts at dst[0, rows*K) and the lo parts right
// after.  valid: entries of M with row (or, transposed, k) index >= valid are zero
// (padding of the vocab-way head).
struct PackJob {
  const float* src;
  void* dst;
  int rows, K, transposed, valid;
};

// The matrices of a model, for pack_kernel: job y < 6 n_layers is matrix y % 6 of
// layer y / 6; the three after them are the vocab-way head, its transpose and the
// plain FP32 transpose.
struct PackPlan {
  const float* theta;
  char* wpack;
  int64_t layer0, layer_stride, qkv_w, ffn1_w, ffn2_w, head_w;
  PackOffsets pk;
  int D, n_layers, vocab;
};

__device__ __forceinline__ PackJob pack_job(const PackPlan& p, int y) {
  const int D = p.D;
  if (y >= 6 * p.n_layers) {
    if (y == 6 * p.n_layers + 2)
      return PackJob{p.theta + p.head_w, p.wpack + p.pk.headF, p.pk.vp, D, 2, p.vocab};
    const bool t = y > 6 * p.n_layers;
    return PackJob{p.theta + p.head_w, p.wpack + (t ? p.pk.headT : p.pk.head), t ? D : p.pk.vp, t ? p.pk.vp : D, t,
                   p.vocab};
  }
  const int l = y / 6, w = y % 6;
  const float* lp = p.theta + p.layer0 + (int64_t)l * p.layer_stride;
  char* wl = p.wpack + (size_t)l * p.pk.layer_stride;
  switch (w) {
    case 0: return PackJob{lp + p.qkv_w, wl + p.pk.qkv, 3 * D, D, 0, 3 * D};
    case 1: return PackJob{lp + p.ffn1_w, wl + p.pk.ffn1, 4 * D, D, 0, 4 * D};
    case 2: return PackJob{lp + p.ffn2_w, wl + p.pk.ffn2, D, 4 * D, 0, D};
    case 3: return PackJob{lp + p.qkv_w, wl + p.pk.qkvT, D, 3 * D, 1, 3 * D};
    case 4: return PackJob{lp + p.ffn1_w, wl + p.pk.ffn1T, D, 4 * D, 1, 4 * D};
    default: return PackJob{lp + p.ffn2_w, wl + p.pk.ffn2T, 4 * D, D, 1, D};
  }
}

// Every matrix in one launch, blockIdx.y = job: a launch per matrix took 4.5 us each
// (60 us of the 676 us training step of a 2-layer, d = 32 model); one launch takes
// 4.3 us there.
template <int MODE>
__global__ void pack_kernel(PackPlan plan) {
  typedef typename Mode<MODE>::WT WT;
  constexpr int KC = Mode<MODE>::KC;
  constexpr int VEC = KC / 4;
  const PackJob j = pack_job(plan, blockIdx.y);
  WT* dst = reinterpret_cast<WT*>(j.dst);
  const int total = j.rows * j.K;
  if (j.transposed == 2) {   // dst[k][r] = src[r][k], FP32
    float* f = reinterpret_cast<float*>(j.dst);
    for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < total; p += gridDim.x * blockDim.x) {
      const int r = p % j.rows, k = p / j.rows;
      f[p] = r < j.valid ? j.src[(size_t)r * j.K + k] : 0.f;
    }
    return;
  }
  const int nchunk = j.K / KC;
  for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < total; p += gridDim.x * blockDim.x) {
    const int e = p % VEC;
    const int pc = p / VEC;
    const int l = pc % 64;
    const int rest = pc / 64;
    const int c = rest % nchunk;
    const int n = rest / nchunk;
    const int r = 16 * n + (l & 15);
    const int k = c * KC + (l >> 4) * VEC + e;
    const float v = j.transposed ? (k < j.valid ? j.src[(size_t)k * j.rows + r] : 0.f)
                                 : (r < j.valid ? j.src[(size_t)r * j.K + k] : 0.f);
    const WT hi = from_f<WT>(v);
    dst[p] = hi;
    if (Mode<MODE>::SPLIT) dst[p + total] = from_f<WT>(v - to_f(hi));
  }
}

template <int MODE>
static hipError_t pack_all(const fvan_model_config& c, const float* theta, void* wpack, hipStream_t s) {
  const ParamOffsets po = param_offsets(c);
  const PackPlan plan{theta,     reinterpret_cast<char*>(wpack), po.layer0, po.layer_stride, po.qkv_w, po.ffn1_w,
                      po.ffn2_w, po.head_w,                       pack_offsets(c), c.d_model, c.n_layers, c.vocab};
  const int jobs = 6 * c.n_layers + (plan.pk.vp ? 3 : 0);
  if (jobs == 0) return hipSuccess;
  const int largest = std::max(4 * c.d_model, plan.pk.vp) * c.d_model;
  hipLaunchKernelGGL((pack_kernel<MODE>), dim3((largest + 255) / 256, jobs), dim3(256), 0, s, plan);
  return hipGetLastError();
}

hipError_t launch_pack(const fvan_model_config& c, const float* theta, void* wpack, hipStream_t s) {
  switch (c.precision) {
    case FVAN_FP32: return pack_all<0>(c, theta, wpack, s);
    case FVAN_BF16_SPLIT: return pack_all<2>(c, theta, wpack, s);
    default: return hipErrorInvalidValue;
  }
}

// Adam (Kingma & Ba) with L2 weight decay folded into the gradient; the
// gradient is zeroed for the next accumulation.
__global__ void adam_kernel(float* __restrict__ theta, float* __restrict__ g, float* __restrict__ m,
                            float* __restrict__ v, int64_t n, float lr, float b1, float b2, float eps, float wd,
                            float c1, float c2) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const float gi = g[i] + wd * theta[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    theta[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    g[i] = 0.0f;
  }
}

hipError_t launch_adam(float* theta, float* grads, float* m, float* v, int64_t n, const fvan_adam& o, int64_t step,
                       hipStream_t s) {
  const double c1 = 1.0 - std::pow((double)o.beta1, (double)step);
  const double c2 = 1.0 - std::pow((double)o.beta2, (double)step);
  const int grid = (int)std::min<int64_t>((n + 255) / 256, 8192);
  hipLaunchKernelGGL(adam_kernel, dim3(grid), dim3(256), 0, s, theta, grads, m, v, n, o.lr, o.beta1, o.beta2, o.eps,
                     o.weight_decay, (float)c1, (float)c2);
  return hipGetLastError();
}

__global__ void zero_int_kernel(int* p, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0;
}

hipError_t launch_zero_int(int* p, int n, hipStream_t s) {
  hipLaunchKernelGGL(zero_int_kernel, dim3(1), dim3(64), 0, s, p, n);
  return hipGetLastError();
}

}  // namespace fvan
