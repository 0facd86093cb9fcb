// Spin energies E_b = - sum_{pairs} J_ij s_i s_j (Eq. 6 for SK, Eq. 8 for EA),
// each unordered pair counted once.
//
// ELL bonds: one workgroup per sample; the sample's int8 spin row is staged in
// LDS with coalesced 16-byte loads, each thread sums its sites' stored pairs
// (neighbour table and bonds are shared by all samples and stay in L2), then a
// fixed-order block reduction.  +/-J bonds accumulate in int32: exact.
// Dense (SK) bonds: one workgroup per 16 samples so every J row read from L2
// serves 16 samples (below).
#include "device_common.h"
#include "fvan_internal.h"

namespace fvan {

constexpr int kEThreads = 256;

template <typename A>
__device__ __forceinline__ A block_sum(A v, A* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) red[wave] = v;
  __syncthreads();
  A r = 0;
  if (threadIdx.x == 0) {
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) r += red[w];
  }
  return r;
}

template <typename JT, typename A>
__global__ __launch_bounds__(kEThreads) void energy_ell_kernel(int n, int deg, const int32_t* __restrict__ nbr,
                                                              const JT* __restrict__ J,
                                                              const int8_t* __restrict__ spins, A* __restrict__ out) {
  extern __shared__ int8_t srow[];
  __shared__ A red[kEThreads / 64];
  const int b = blockIdx.x;
  const int8_t* row = spins + (size_t)b * n;
  // stage the row: 16-byte loads where aligned, bytes for the tail
  const int n16 = ((((uintptr_t)row) & 15) == 0) ? (n >> 4) : 0;
  for (int i = threadIdx.x; i < n16; i += kEThreads)
    reinterpret_cast<uint4*>(srow)[i] = reinterpret_cast<const uint4*>(row)[i];
  for (int i = n16 * 16 + threadIdx.x; i < n; i += kEThreads) srow[i] = row[i];
  __syncthreads();
  A acc = 0;
  for (int i = threadIdx.x; i < n; i += kEThreads) {
    const A si = (A)srow[i];
    A part = 0;
    for (int k = 0; k < deg; ++k) {
      const int j = nbr[(size_t)i * deg + k];
      if (j >= 0 && j < n) part += (A)J[(size_t)i * deg + k] * (A)srow[j];
    }
    acc += si * part;
  }
  const A tot = block_sum<A>(acc, red);
  if (threadIdx.x == 0) out[b] = -tot;
}

// Dense (SK) bonds.  One workgroup (4 waves) per kDenseS samples; wave w takes the
// rows i = w, w + 4, ... of J, lane l the columns j = l, l + 64, ..., and every J
// element a lane loads serves all the samples:
//   acc += J_ij (s_i s_j), rows in order, then a fixed-order block sum.
// energy_dense_general_kernel forms s_i s_j from LDS for every (i, j, sample).
//
// For +-1 spins acc is carried multiplied by s_i instead: s_i (acc + J_ij s_i s_j) =
// s_i acc + J_ij s_j with the same roundings (a sign flip is exact), so a row costs
// one FMA per element with the lane's s_j held in registers, and one sign flip per
// row and sample.  That is the vector FMA rate (2 B n^2 flop at 78 TFLOP/s without
// packed FP32: 55 us at 8192 x 512).  Measured there: 331 us with the product formed
// per element, 77 us now.  (FP32 MFMA takes 50 us in another summation order, but
// the weights of a training step then differ in the last bit, which the sampling of
// the next step amplifies into other spins.)
constexpr int kDenseS = 16;

__global__ __launch_bounds__(kEThreads) void energy_dense_general_kernel(int n, int batch, const float* __restrict__ J,
                                                                         const int8_t* __restrict__ spins,
                                                                         float* __restrict__ out) {
  extern __shared__ int8_t sm[];    // [kDenseS][n]
  __shared__ float red[kEThreads / 64];
  const int b0 = blockIdx.x * kDenseS;
  const int ns = min(kDenseS, batch - b0);
  for (int i = threadIdx.x; i < kDenseS * n; i += kEThreads) {
    const int s = i / n, j = i % n;
    sm[i] = s < ns ? spins[(size_t)(b0 + s) * n + j] : (int8_t)0;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float acc[kDenseS];
#pragma unroll
  for (int s = 0; s < kDenseS; ++s) acc[s] = 0.f;
  for (int i = wave; i < n; i += kEThreads / 64) {
    const float* Ji = J + (size_t)i * n;
    for (int j = lane; j < n; j += 64) {
      const float w = Ji[j];
#pragma unroll
      for (int s = 0; s < kDenseS; ++s) acc[s] += w * (float)(sm[s * n + i] * sm[s * n + j]);
    }
  }
  for (int s = 0; s < kDenseS; ++s) {
    const float tot = block_sum<float>(acc[s], red);
    if (threadIdx.x == 0 && s < ns) out[b0 + s] = -0.5f * tot;
    __syncthreads();
  }
}

// 12 < n <= 64 NJ, any spins (a workgroup that finds one that is not +-1 takes the
// products as the general kernel does).
template <int NJ>
__global__ __launch_bounds__(kEThreads) void energy_dense_kernel(int n, int batch, const float* __restrict__ J,
                                                                 const int8_t* __restrict__ spins,
                                                                 float* __restrict__ out) {
  constexpr int NP = 64 * NJ;                // columns, padded
  __shared__ __align__(16) int8_t sm[kDenseS][NP];   // the tile's spins (absent samples 0, columns past n 1)
  __shared__ uint32_t up[NP];                // bit s: sample s of the tile has spin +1 at site i
  __shared__ float red[kEThreads / 64];
  const int b0 = blockIdx.x * kDenseS;
  const int ns = min(kDenseS, batch - b0);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int8_t* base = spins + (size_t)b0 * n;
  if (n == NP && ((uintptr_t)base & 15) == 0) {
    constexpr int V = kDenseS * NP / 16;     // 16-byte pieces of the tile, whole rows
#pragma unroll
    for (int x0 = 0; x0 < V; x0 += kEThreads) {
      const int x = x0 + threadIdx.x;
      if (x < V)
        reinterpret_cast<uint4*>(&sm[0][0])[x] =
            x < ns * (NP / 16) ? reinterpret_cast<const uint4*>(base)[x] : make_uint4(0u, 0u, 0u, 0u);
    }
  } else {
#pragma unroll 8
    for (int x = threadIdx.x; x < kDenseS * NP; x += kEThreads) {
      const int s = x / NP, j = x % NP;
      const int8_t v = base[min(s, ns - 1) * n + min(j, n - 1)];
      sm[s][j] = j >= n ? (int8_t)1 : s < ns ? v : (int8_t)0;
    }
  }
  __syncthreads();
  float sj[NJ][kDenseS];                     // the lane's spins
  int odd = 0;                               // nonzero if one of them is not +-1
#pragma unroll
  for (int q = 0; q < NJ; ++q)
#pragma unroll
    for (int s = 0; s < kDenseS; ++s) {
      const int v = sm[s][lane + 64 * q];
      odd |= s < ns ? v * v - 1 : 0;
      sj[q][s] = (float)v;
    }
  for (int i = threadIdx.x; i < NP; i += kEThreads) {
    uint32_t m = 0;
#pragma unroll
    for (int s = 0; s < kDenseS; ++s) m |= (sm[s][i] > 0 ? 1u : 0u) << s;
    up[i] = m;
  }
  const bool all_pm1 = !__syncthreads_or(odd);
  float acc[kDenseS];
#pragma unroll
  for (int s = 0; s < kDenseS; ++s) acc[s] = 0.f;
  if (all_pm1) {
    uint32_t prev = 0xFFFFFFFFu;             // signs acc is carried with: +1 at first
    float w[NJ];
    auto load = [&](int i, float* v) {
#pragma unroll
      for (int q = 0; q < NJ; ++q) {
        const int j = lane + 64 * q;
        const float x = J[(size_t)min(i, n - 1) * n + min(j, n - 1)];   // no branch around the load
        v[q] = j < n ? x : 0.f;
      }
    };
    load(wave, w);
    for (int i = wave; i < n; i += kEThreads / 64) {
      float nw[NJ];
      load(i + kEThreads / 64, nw);          // the wave's next row, in flight during this one
      const uint32_t cur = __builtin_amdgcn_readfirstlane(up[i]), flip = cur ^ prev;
      prev = cur;
#pragma unroll
      for (int s = 0; s < kDenseS; ++s)
        acc[s] = __uint_as_float(__float_as_uint(acc[s]) ^ ((flip >> s & 1u) << 31));
#pragma unroll
      for (int q = 0; q < NJ; ++q)
#pragma unroll
        for (int s = 0; s < kDenseS; ++s) acc[s] += w[q] * sj[q][s];
#pragma unroll
      for (int q = 0; q < NJ; ++q) w[q] = nw[q];
    }
#pragma unroll
    for (int s = 0; s < kDenseS; ++s) acc[s] = prev >> s & 1u ? acc[s] : -acc[s];
  } else {
    for (int i = wave; i < n; i += kEThreads / 64)
#pragma unroll
      for (int q = 0; q < NJ; ++q) {
        const int j = lane + 64 * q;
        if (j >= n) continue;
        const float w = J[(size_t)i * n + j];
#pragma unroll
        for (int s = 0; s < kDenseS; ++s)
          acc[s] += w * (float)((int)sm[s][i] * (int)sm[s][j]);
      }
  }
  for (int s = 0; s < kDenseS; ++s) {
    const float tot = block_sum<float>(acc[s], red);
    if (threadIdx.x == 0 && s < ns) out[b0 + s] = -0.5f * tot;
    __syncthreads();
  }
}

static void launch_dense(int n, int batch, const float* J, const int8_t* spins, float* out, hipStream_t s) {
  const dim3 grid((batch + kDenseS - 1) / kDenseS);
  // n > 512: a lane's spins no longer fit its registers.  n <= 12: the rows are too few to
  // pay for staging 64 columns (30000 samples of 1, 8, 12 and 16 spins: 14.7, 16.4, 18.0 and
  // 19.0 us with the general kernel, 16.5, 17.4, 18.0 and 18.5 with the registers).
  if (n <= 12 || n > 512) {
    hipLaunchKernelGGL(energy_dense_general_kernel, grid, dim3(kEThreads), kDenseS * n, s, n, batch, J, spins, out);
    return;
  }
  auto kern = n <= 64 ? energy_dense_kernel<1> : n <= 128 ? energy_dense_kernel<2> : n <= 256 ? energy_dense_kernel<4>
                                                                                     : energy_dense_kernel<8>;
  hipLaunchKernelGGL(kern, grid, dim3(kEThreads), 0, s, n, batch, J, spins, out);
}

hipError_t launch_energy(const fvan_couplings& c, int32_t batch, const int8_t* spins, void* energy,
                         hipStream_t s) {
  const int n = c.n_spins;
  if (c.kind == FVAN_BONDS_PM1) {
    hipLaunchKernelGGL((energy_ell_kernel<int8_t, int>), dim3(batch), dim3(kEThreads), n, s, n, c.degree, c.nbr,
                       (const int8_t*)c.J, spins, (int*)energy);
  } else if (c.kind == FVAN_BONDS_F32) {
    hipLaunchKernelGGL((energy_ell_kernel<float, float>), dim3(batch), dim3(kEThreads), n, s, n, c.degree, c.nbr,
                       (const float*)c.J, spins, (float*)energy);
  } else {
    launch_dense(n, batch, (const float*)c.J, spins, (float*)energy, s);
  }
  return hipGetLastError();
}

}  // namespace fvan
