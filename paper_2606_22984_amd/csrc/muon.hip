// Muon update (Methods, comparison of optimisers): momentum, Newton-Schulz
// orthogonalisation of the momentum matrix on FP32 MFMA, and the scaled step
// with decoupled weight decay; the parameters that are not layer weight
// matrices take Adam in the same call.
//
// The matrix is iterated in place, viewed as the wide matrix Z (m x n, m =
// min(rows, cols) <= 128): a tall matrix is read through transposed strides.  Per
// iteration:
//   Gram     A = Z Z^T           upper-triangle 16x16 tiles, mirrored
//   poly     P = b A + c A A     LDS -> LDS (A A is symmetric: same mirroring)
//   update   Z <- a Z + P Z      each wave owns 16-column blocks of Z; it holds
//                                its block's K fragments in registers before
//                                it overwrites the block
// with (a, b, c) = (3.4445, -4.7750, 2.0315), the quintic coefficients
// published with the Muon optimiser.  All products are FP32 MFMA 16x16x4 with FP32
// accumulation.  Where Z lives and how many workgroups share a matrix goes by size:
//   m <= 64   one 8-wave workgroup per matrix, Z in LDS for the whole update
//             (muon_kernel).  With Z in global memory and one element of each
//             array in flight: 60 us (d = 32, 2 layers) and 291 us (d = 64, 4
//             layers); now 18 us and 68 us
//   m = 128   Z (up to 256 KB) does not fit a compute unit: one launch per phase,
//             the Gram matrix as one wave per 16x16 tile, the update as one
//             workgroup per 64 columns (muon_begin / scale / gram / update
//             kernels).  One workgroup per matrix waited on L2 for its Gram
//             operands: 1.78 ms for two layers' matrices, 0.21 ms now
// Every form adds the products in the same order.  The norm of the momentum, in FP64, is
// one workgroup's sum up to m = 64 and 32 workgroups' sums at m = 128.
// The standalone orthogonalisation (no workspace) is one workgroup with Z in
// global memory.
#include <cmath>

#include "device_common.h"
#include "fvan_internal.h"

namespace fvan {

constexpr int kNsMaxGram = 128;          // largest min(rows, cols)
constexpr int kNsThreads = 512;          // 8 waves
constexpr int kNsWaves = kNsThreads / 64;
constexpr float kNsA = 3.4445f, kNsB = -4.7750f, kNsC = 2.0315f;

template <int MG>                        // largest m
struct NsSmem {
  float gram[MG][MG + 4];                // row pitch 4 mod 64: conflict-free fragment reads
  float poly[MG][MG + 4];
  double part[kNsWaves];
};

// Z(i, j) = p[i * si + j * sj], 0 <= i < m <= n, 0 <= j < n.
struct ZView {
  float* p;
  int m, n;
  int64_t si, sj;
};

__device__ __forceinline__ ZView wide_view(float* p, int rows, int cols) {
  if (rows <= cols) return ZView{p, rows, cols, (int64_t)cols, 1};
  return ZView{p, cols, rows, 1, (int64_t)cols};
}

__device__ __forceinline__ floatx4 mfma4(float a, float b, floatx4 acc) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0);
}

// p-th pair (ti, tj), ti <= tj, of mt x mt tiles in row-major upper-triangle order.
__device__ __forceinline__ void upper_pair(int p, int mt, int& ti, int& tj) {
  ti = 0;
  while (p >= mt - ti) {
    p -= mt - ti;
    ++ti;
  }
  tj = ti + p;
}

// Sum of v over the workgroup in a fixed order (bitwise reproducible).
template <int MG>
__device__ double block_sum(double v, NsSmem<MG>& sm) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) sm.part[wave] = v;
  __syncthreads();
  double s = 0.0;
  for (int w = 0; w < kNsWaves; ++w) s += sm.part[w];
  __syncthreads();
  return s;
}

// P = b A + c A A from the Gram matrix in sm.gram (symmetric: upper tiles, mirrored).
// FULL: the matrix fills MG (the K loop is unrolled, so the LDS reads of several
// steps are in flight).
template <int MG, bool FULL = false>
__device__ __forceinline__ void ns_poly(NsSmem<MG>& sm, int mt) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r16 = lane & 15, g = lane >> 4;
  const int npairs = mt * (mt + 1) / 2;
  for (int p = wave; p < npairs; p += kNsWaves) {
    int ti, tj;
    upper_pair(p, mt, ti, tj);
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    auto step = [&](int k) { acc = mfma4(sm.gram[16 * ti + r16][k + g], sm.gram[k + g][16 * tj + r16], acc); };
    if constexpr (FULL) {
#pragma unroll
      for (int k = 0; k < MG; k += 4) step(k);
    } else {
      for (int t = 0; t < mt; ++t)         // 16 of K at a time
#pragma unroll
        for (int u = 0; u < 4; ++u) step(16 * t + 4 * u);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = 16 * ti + 4 * g + i, col = 16 * tj + r16;
      const float v = kNsB * sm.gram[row][col] + kNsC * acc[i];
      sm.poly[row][col] = v;
      if (ti != tj) sm.poly[col][row] = v;
    }
  }
}

// steps Newton-Schulz iterations on Z in place (Z already normalised).
// FULL: z.m == MG and z.n is a multiple of 16 (no edges, K loops unrolled).
template <int MG, bool FULL = false>
__device__ __forceinline__ void ns_iterate(const ZView z, int steps, NsSmem<MG>& sm) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r16 = lane & 15, g = lane >> 4;
  const int mt = FULL ? MG / 16 : (z.m + 15) >> 4;
  const int kg = 4 * mt;                 // K steps of 4 over the padded Gram dimension
  const int npairs = mt * (mt + 1) / 2;
  const int nb = (z.n + 15) >> 4;
  for (int it = 0; it < steps; ++it) {
    // ---- A = Z Z^T: lane supplies A-operand Z(16ti + r16, k) and B-operand Z(16tj + r16, k), k = k0 + g
    for (int p = wave; p < npairs; p += kNsWaves) {
      int ti, tj;
      upper_pair(p, mt, ti, tj);
      const int ia = 16 * ti + r16, ib = 16 * tj + r16;
      const float* za = z.p + (int64_t)min(ia, z.m - 1) * z.si;
      const float* zb = z.p + (int64_t)min(ib, z.m - 1) * z.si;
      const bool va = FULL || ia < z.m, vb = FULL || ib < z.m;
      floatx4 acc = {0.f, 0.f, 0.f, 0.f};
      int k0 = 0;
      for (; k0 + 16 <= z.n; k0 += 16) {
        float a[4], b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int64_t o = (int64_t)(k0 + 4 * u + g) * z.sj;
          a[u] = va ? za[o] : 0.f;
          b[u] = vb ? zb[o] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) acc = mfma4(a[u], b[u], acc);
      }
      for (; !FULL && k0 < z.n; k0 += 4) {
        const int k = k0 + g;
        const int64_t o = (int64_t)min(k, z.n - 1) * z.sj;
        const float a = (va && k < z.n) ? za[o] : 0.f;
        const float b = (vb && k < z.n) ? zb[o] : 0.f;
        acc = mfma4(a, b, acc);
      }
      // lane holds A(16ti + 4g + i, 16tj + r16)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = 16 * ti + 4 * g + i, col = 16 * tj + r16;
        sm.gram[row][col] = acc[i];
        if (ti != tj) sm.gram[col][row] = acc[i];
      }
    }
    __syncthreads();
    ns_poly<MG, FULL>(sm, mt);
    __syncthreads();
    // ---- Z <- a Z + P Z, one 16-column block per wave at a time
    for (int jb = wave; jb < nb; jb += kNsWaves) {
      const int j = 16 * jb + r16;
      const bool vj = FULL || j < z.n;
      float* zc = z.p + (int64_t)min(j, z.n - 1) * z.sj;
      float zf[MG / 4];                  // Z(4s + g, j)
#pragma unroll
      for (int s = 0; s < MG / 4; ++s) {
        const int k = 4 * s + g;
        zf[s] = FULL || (s < kg && vj && k < z.m) ? zc[(int64_t)k * z.si] : 0.f;
      }
      for (int ti = 0; ti < mt; ++ti) {
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < MG / 4; ++s)
          if (s < kg) acc = mfma4(sm.poly[16 * ti + r16][4 * s + g], zf[s], acc);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = 16 * ti + 4 * g + i;
          if (FULL || (vj && row < z.m)) {
            float* q = zc + (int64_t)row * z.si;
            *q = kNsA * *q + acc[i];
          }
        }
      }
    }
    __syncthreads();
  }
}

// Standalone orthogonalisation: O = NewtonSchulz(M), O may alias M.
__global__ void __launch_bounds__(kNsThreads) newton_schulz_kernel(const float* M, float* O, int rows, int cols,
                                                                   int steps, float eps) {
  __shared__ NsSmem<kNsMaxGram> sm;
  const int64_t total = (int64_t)rows * cols;
  double ss = 0.0;
  for (int64_t i = threadIdx.x; i < total; i += kNsThreads) {
    const float v = M[i];
    O[i] = v;
    ss += (double)v * v;
  }
  const float inv = (float)(1.0 / (sqrt(block_sum(ss, sm)) + (double)eps));
  for (int64_t i = threadIdx.x; i < total; i += kNsThreads) O[i] *= inv;
  __syncthreads();
  ns_iterate(wide_view(O, rows, cols), steps, sm);
}

// Offsets of the three weight matrices inside each layer's parameter block.
struct MuonLayout {
  int64_t layer0, stride;
  int64_t off[3];
  int rows[3], cols[3];
  int n_layers;
};

__device__ __forceinline__ bool in_muon_matrix(int64_t i, const MuonLayout& L) {
  if (i < L.layer0 || i >= L.layer0 + L.n_layers * L.stride) return false;
  const int64_t o = (i - L.layer0) % L.stride;
#pragma unroll
  for (int w = 0; w < 3; ++w)
    if (o >= L.off[w] && o < L.off[w] + (int64_t)L.rows[w] * L.cols[w]) return true;
  return false;
}

// The step W -= lr (scale O + wd W), scale = rms_scale sqrt(max(rows, cols)).
__device__ __forceinline__ float muon_stepped(float w, float o, float lr, float scale, float wd) {
  return w - lr * (scale * o + wd * w);
}

// d = MG <= 64.  Workgroup (layer, which): momentum, orthogonalisation of Z in
// LDS, step, and the gradient cleared for the next accumulation.
template <int MG>
__global__ void __launch_bounds__(kNsThreads) muon_kernel(float* __restrict__ theta, float* __restrict__ grads,
                                                          float* __restrict__ mom, MuonLayout L, float lr, float mu,
                                                          float wd, float rms_scale, float eps, int steps) {
  constexpr int PZ = 4 * MG + 4;             // row pitch of Z: 4 mod 64
  __shared__ NsSmem<MG> sm;
  __shared__ float zs[MG][PZ];
  const int layer = blockIdx.x / 3, w = blockIdx.x % 3;
  const int rows = L.rows[w], cols = L.cols[w];
  const int64_t base = L.layer0 + layer * L.stride + L.off[w];
  float* W = theta + base;
  float* Gm = grads + base;
  float* Mm = mom + base;
  const int total = rows * cols;             // a multiple of kNsThreads (d is 32 or 64)
  const bool tall = rows > cols;             // element (r, c) is Z(c, r)
  const int cs = __builtin_ctz(cols);        // cols is a power of two
  auto at = [&](int i) -> float& {
    const int r = i >> cs, c = i & (cols - 1);
    return tall ? zs[c][r] : zs[r][c];
  };
  // eight elements of each array in flight per thread: one at a time, these two
  // passes took most of the kernel
  constexpr int U = 8;
  double ss = 0.0;
  for (int i0 = threadIdx.x; i0 < total; i0 += U * kNsThreads) {
    float mv[U], gv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = min(i0 + u * kNsThreads, total - 1);
      mv[u] = Mm[i];
      gv[u] = Gm[i];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * kNsThreads;
      if (i < total) {
        const float v = mu * mv[u] + gv[u];
        Mm[i] = v;
        at(i) = v;
        ss += (double)v * v;
      }
    }
  }
  const float inv = (float)(1.0 / (sqrt(block_sum(ss, sm)) + (double)eps));
  const int n = max(rows, cols);
  for (int i = threadIdx.x; i < total; i += kNsThreads) at(i) *= inv;
  __syncthreads();
  ns_iterate<MG, true>(ZView{&zs[0][0], MG, n, PZ, 1}, steps, sm);
  const float scale = rms_scale * sqrtf((float)n);
  for (int i0 = threadIdx.x; i0 < total; i0 += U * kNsThreads) {
    float wv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) wv[u] = W[min(i0 + u * kNsThreads, total - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * kNsThreads;
      if (i < total) {
        W[i] = muon_stepped(wv[u], at(i), lr, scale, wd);
        Gm[i] = 0.0f;
      }
    }
  }
}

// ---- d = 128: the same update, a phase per launch ----
// blockIdx.y is the matrix (layer, which).  The momentum replaces the gradient,
// which Newton-Schulz then iterates in place; partial sums of its squares per
// workgroup of muon_begin_kernel, in FP64.
constexpr int kMuonBlocks = 32;
struct MuonMatrix {
  int64_t base;
  int rows, cols;
};
__device__ __forceinline__ MuonMatrix muon_matrix(const MuonLayout& L, int y) {
  const int layer = y / 3, w = y % 3;
  return MuonMatrix{L.layer0 + layer * L.stride + L.off[w], L.rows[w], L.cols[w]};
}

__global__ void __launch_bounds__(256) muon_begin_kernel(float* __restrict__ grads, float* __restrict__ mom,
                                                         MuonLayout L, float mu, double* __restrict__ part) {
  __shared__ double red[4];
  const MuonMatrix x = muon_matrix(L, blockIdx.y);
  float* G = grads + x.base;
  float* M = mom + x.base;
  const int total = x.rows * x.cols;
  double ss = 0.0;
#pragma unroll 4
  for (int i = blockIdx.x * 256 + threadIdx.x; i < total; i += kMuonBlocks * 256) {
    const float v = mu * M[i] + G[i];
    M[i] = v;
    G[i] = v;
    ss += (double)v * v;
  }
  for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.y * kMuonBlocks + blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

__global__ void __launch_bounds__(256) muon_scale_kernel(float* __restrict__ grads, MuonLayout L, float eps,
                                                         const double* __restrict__ part) {
  const MuonMatrix x = muon_matrix(L, blockIdx.y);
  double ss = part[blockIdx.y * kMuonBlocks + (threadIdx.x & (kMuonBlocks - 1))];
  for (int off = kMuonBlocks / 2; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
  const float inv = (float)(1.0 / (sqrt(ss) + (double)eps));
  const int total = x.rows * x.cols;
#pragma unroll 4
  for (int i = blockIdx.x * 256 + threadIdx.x; i < total; i += kMuonBlocks * 256) grads[x.base + i] *= inv;
}

// A = Z Z^T, one wave per upper-triangle 16x16 tile (summed over n in one chain, in
// the order of ns_iterate), 32 columns' operands in flight.
__global__ void __launch_bounds__(64) muon_gram_kernel(float* __restrict__ grads, MuonLayout L,
                                                       float* __restrict__ gram) {
  constexpr int MG = kNsMaxGram;
  const MuonMatrix x = muon_matrix(L, blockIdx.y);
  const ZView z = wide_view(grads + x.base, x.rows, x.cols);
  const int lane = threadIdx.x, r16 = lane & 15, g = lane >> 4;
  int ti, tj;
  upper_pair(blockIdx.x, MG / 16, ti, tj);
  const float* za = z.p + (16 * ti + r16) * z.si + g * z.sj;
  const float* zb = z.p + (16 * tj + r16) * z.si + g * z.sj;
  constexpr int U = 8;                       // K steps of 4 per round; n = 384 or 512
  float a[U], b[U];
  auto load = [&](int k0, float* p, float* q) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      p[u] = za[(k0 + 4 * u) * z.sj];
      q[u] = zb[(k0 + 4 * u) * z.sj];
    }
  };
  load(0, a, b);
  floatx4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < z.n; k0 += 4 * U) {
    float an[U], bn[U];
    if (k0 + 4 * U < z.n) load(k0 + 4 * U, an, bn);
#pragma unroll
    for (int u = 0; u < U; ++u) acc = mfma4(a[u], b[u], acc);
#pragma unroll
    for (int u = 0; u < U; ++u) { a[u] = an[u]; b[u] = bn[u]; }
  }
  float* A = gram + (size_t)blockIdx.y * MG * MG;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = 16 * ti + 4 * g + i, col = 16 * tj + r16;
    A[row * MG + col] = acc[i];
    if (ti != tj) A[col * MG + row] = acc[i];
  }
}

// P from the Gram matrix (every workgroup of a matrix forms it, 2 us) and
// Z <- a Z + P Z for 64 columns: wave w takes the 16-column block w % 4 and half of
// the rows.  last: the step on W from the finished O instead, and the gradient cleared.
__global__ void __launch_bounds__(kNsThreads) muon_update_kernel(float* __restrict__ theta, float* __restrict__ grads,
                                                                 MuonLayout L, const float* __restrict__ gram, int last,
                                                                 float lr, float wd, float rms_scale) {
  constexpr int MG = kNsMaxGram, MT = MG / 16;
  __shared__ NsSmem<MG> sm;
  const MuonMatrix x = muon_matrix(L, blockIdx.y);
  const ZView z = wide_view(grads + x.base, x.rows, x.cols);
  if (64 * (int)blockIdx.x >= z.n) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r16 = lane & 15, g = lane >> 4;
  const int64_t j = 64 * blockIdx.x + 16 * (wave & 3) + r16;
  float zf[MG / 4];                          // Z(4s + g, j)
#pragma unroll
  for (int s = 0; s < MG / 4; ++s) zf[s] = z.p[(4 * s + g) * z.si + j * z.sj];
  const float* A = gram + (size_t)blockIdx.y * MG * MG;
#pragma unroll
  for (int i = 0; i < MG * MG / 4; i += kNsThreads) {
    const int e = (i + (int)threadIdx.x) * 4;
    *reinterpret_cast<float4*>(&sm.gram[e / MG][e % MG]) = *reinterpret_cast<const float4*>(A + e);
  }
  __syncthreads();
  ns_poly<MG, true>(sm, MT);
  __syncthreads();                           // P is formed; every wave holds its columns of Z
  floatx4 acc[MT / 2];
#pragma unroll
  for (int t = 0; t < MT / 2; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int t0 = (wave >> 2) * (MT / 2);
#pragma unroll
  for (int s = 0; s < MG / 4; ++s)
#pragma unroll
    for (int t = 0; t < MT / 2; ++t) acc[t] = mfma4(sm.poly[16 * (t0 + t) + r16][4 * s + g], zf[s], acc[t]);
  const float scale = rms_scale * sqrtf((float)z.n);
#pragma unroll
  for (int t = 0; t < MT / 2; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t o = (16 * (t0 + t) + 4 * g + i) * z.si + j * z.sj;
      const float v = kNsA * z.p[o] + acc[t][i];
      if (last) {
        float* W = theta + x.base;
        W[o] = muon_stepped(W[o], v, lr, scale, wd);
        z.p[o] = 0.0f;
      } else {
        z.p[o] = v;
      }
    }
}

// No iterations: the step from the normalised momentum.
__global__ void __launch_bounds__(256) muon_step_kernel(float* __restrict__ theta, float* __restrict__ grads,
                                                        MuonLayout L, float lr, float wd, float rms_scale) {
  const MuonMatrix x = muon_matrix(L, blockIdx.y);
  const float scale = rms_scale * sqrtf((float)max(x.rows, x.cols));
  const int total = x.rows * x.cols;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < total; i += kMuonBlocks * 256) {
    theta[x.base + i] = muon_stepped(theta[x.base + i], grads[x.base + i], lr, scale, wd);
    grads[x.base + i] = 0.0f;
  }
}

// Adam on the parameters outside the layer weight matrices; same update as
// the library's Adam step.
__global__ void adam_rest_kernel(float* __restrict__ theta, float* __restrict__ g, float* __restrict__ m,
                                 float* __restrict__ v, int64_t n, MuonLayout L, float lr, float b1, float b2,
                                 float eps, float wd, float c1, float c2) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    if (in_muon_matrix(i, L)) continue;
    const float gi = g[i] + wd * theta[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    theta[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    g[i] = 0.0f;
  }
}

hipError_t launch_newton_schulz(const float* M, float* O, int rows, int cols, int steps, float eps, hipStream_t s) {
  if (rows < 1 || cols < 1 || (rows < cols ? rows : cols) > kNsMaxGram) return hipErrorInvalidValue;
  hipLaunchKernelGGL(newton_schulz_kernel, dim3(1), dim3(kNsThreads), 0, s, M, O, rows, cols, steps, eps);
  return hipGetLastError();
}

hipError_t launch_muon(const fvan_model_config& c, float* theta, float* grads, float* m, float* v, int64_t n,
                       const fvan_muon& o, int64_t step, float* scratch, hipStream_t s) {
  const ParamOffsets po = param_offsets(c);
  const int d = c.d_model;
  if (d > kNsMaxGram) return hipErrorInvalidValue;
  MuonLayout L{};
  L.layer0 = po.layer0;
  L.stride = po.layer_stride;
  L.n_layers = c.n_layers;
  L.off[0] = po.qkv_w;  L.rows[0] = 3 * d; L.cols[0] = d;
  L.off[1] = po.ffn1_w; L.rows[1] = 4 * d; L.cols[1] = d;
  L.off[2] = po.ffn2_w; L.rows[2] = d;     L.cols[2] = 4 * d;
  const double c1 = 1.0 - std::pow((double)o.adam.beta1, (double)step);
  const double c2 = 1.0 - std::pow((double)o.adam.beta2, (double)step);
  const int grid = (int)std::min<int64_t>((n + 255) / 256, 8192);
  hipLaunchKernelGGL(adam_rest_kernel, dim3(grid), dim3(256), 0, s, theta, grads, m, v, n, L, o.adam.lr,
                     o.adam.beta1, o.adam.beta2, o.adam.eps, o.adam.weight_decay, (float)c1, (float)c2);
  const int mats = 3 * c.n_layers;
  if (mats == 0) return hipGetLastError();
  if (d <= 64) {
    auto kern = d <= 32 ? muon_kernel<32> : muon_kernel<64>;
    hipLaunchKernelGGL(kern, dim3(mats), dim3(kNsThreads), 0, s, theta, grads, m, L, o.lr, o.momentum, o.weight_decay,
                       o.rms_scale, o.ns_eps, o.ns_steps);
    return hipGetLastError();
  }
  if (d != kNsMaxGram || !scratch) return hipErrorInvalidValue;
  double* part = reinterpret_cast<double*>(scratch);
  float* gram = scratch + 2 * (size_t)mats * kMuonBlocks;
  const dim3 flat(kMuonBlocks, mats);
  hipLaunchKernelGGL(muon_begin_kernel, flat, dim3(256), 0, s, grads, m, L, o.momentum, part);
  hipLaunchKernelGGL(muon_scale_kernel, flat, dim3(256), 0, s, grads, L, o.ns_eps, (const double*)part);
  constexpr int kPairs = kNsMaxGram / 16 * (kNsMaxGram / 16 + 1) / 2;
  for (int it = 0; it < o.ns_steps; ++it) {
    hipLaunchKernelGGL(muon_gram_kernel, dim3(kPairs, mats), dim3(64), 0, s, grads, L, gram);
    hipLaunchKernelGGL(muon_update_kernel, dim3(4 * d / 64, mats), dim3(kNsThreads), 0, s, theta, grads, L,
                       (const float*)gram, it + 1 == o.ns_steps ? 1 : 0, o.lr, o.weight_decay, o.rms_scale);
  }
  if (o.ns_steps == 0)
    hipLaunchKernelGGL(muon_step_kernel, flat, dim3(256), 0, s, theta, grads, L, o.lr, o.weight_decay, o.rms_scale);
  return hipGetLastError();
}

}  // namespace fvan
