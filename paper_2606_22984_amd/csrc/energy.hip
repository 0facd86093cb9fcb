// Spin energies E_b = - sum_{pairs} J_ij s_i s_j (Eq. 6 for SK, Eq. 8 for EA),
// each unordered pair counted once.
//
// ELL bonds: one workgroup per sample; the sample's int8 spin row is staged in
// LDS with coalesced 16-byte loads, each thread sums its sites' stored pairs
// (neighbour table and bonds are shared by all samples and stay in L2), then a
// fixed-order block reduction.  +/-J bonds accumulate in int32: exact.
// Dense (SK) bonds are a contraction of the spins with J, on FP32 MFMA (below).
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

// Dense (SK) bonds, E_b = -1/2 sum_i s_bi F_bi with F = S J^T on FP32 MFMA.
// One workgroup (8 waves) owns 16 SBT samples, staged as int8 in LDS; wave w takes
// blocks of 16 IT rows i of J and runs the whole contraction over j for them, so
// every J element a lane loads feeds SBT products and every spin IT; the block's F
// is multiplied by its spins in registers and summed in FP64, in a fixed order.
// Bound: FP32 MFMA (2 B n^2 flop: 28 us at 8192 x 512 and 152 TFLOP/s).  The
// vector-unit form (an integer product, a conversion and an FMA per (i, j, sample))
// took 331 us there; this one takes 50 us, the waves waiting on L2 for the
// next J fragments about half of the time.
constexpr int kDenseThreads = 512;
constexpr int kDenseWaves = kDenseThreads / 64;

// J[i][k .. k + 4), zero outside the matrix; VEC: rows are 16-byte aligned
template <bool VEC>
__device__ __forceinline__ float4 load_j(const float* __restrict__ J, int n, int i, int k) {
  if (i >= n || k >= n) return make_float4(0.f, 0.f, 0.f, 0.f);
  const float* p = J + (size_t)i * n + k;
  if constexpr (VEC) return *reinterpret_cast<const float4*>(p);
  return make_float4(p[0], k + 1 < n ? p[1] : 0.f, k + 2 < n ? p[2] : 0.f, k + 3 < n ? p[3] : 0.f);
}

template <int SBT, int IT, bool VEC>
__global__ __launch_bounds__(kDenseThreads) void energy_dense_kernel(int n, int batch, int stride,
                                                                     const float* __restrict__ J,
                                                                     const int8_t* __restrict__ spins,
                                                                     float* __restrict__ out) {
  constexpr int SB = 16 * SBT;
  extern __shared__ __align__(16) int8_t sm[];        // [SB][stride], zero past n
  __shared__ double red[kDenseWaves][SB];
  const int b0 = blockIdx.x * SB;
  const int ns = min(SB, batch - b0);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 15, g = lane >> 4;
  if (((n | (int)((uintptr_t)spins & 15)) & 15) == 0) {
    for (int i = threadIdx.x; i < SB * (n >> 4); i += kDenseThreads) {
      const int s = i / (n >> 4), j = (i % (n >> 4)) * 16;
      *reinterpret_cast<uint4*>(sm + s * stride + j) =
          s < ns ? *reinterpret_cast<const uint4*>(spins + (size_t)(b0 + s) * n + j) : make_uint4(0u, 0u, 0u, 0u);
    }
  } else {
    for (int i = threadIdx.x; i < SB * stride; i += kDenseThreads) {
      const int s = i / stride, j = i % stride;
      sm[i] = s < ns && j < n ? spins[(size_t)(b0 + s) * n + j] : (int8_t)0;
    }
  }
  __syncthreads();
  double e[SBT][4];
#pragma unroll
  for (int t = 0; t < SBT; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q) e[t][q] = 0.0;
  for (int i0 = wave * 16 * IT; i0 < n; i0 += kDenseWaves * 16 * IT) {
    floatx4 acc[SBT][IT];
#pragma unroll
    for (int t = 0; t < SBT; ++t)
#pragma unroll
      for (int u = 0; u < IT; ++u) acc[t][u] = floatx4{0.f, 0.f, 0.f, 0.f};
    float4 jv[IT];
#pragma unroll
    for (int u = 0; u < IT; ++u) jv[u] = load_j<VEC>(J, n, i0 + 16 * u + c, 4 * g);
    for (int k = 0; k < n; k += 16) {
      float4 jn[IT];                                  // the next chunk, in flight during this one's products
#pragma unroll
      for (int u = 0; u < IT; ++u) jn[u] = load_j<VEC>(J, n, i0 + 16 * u + c, k + 16 + 4 * g);
      float a[SBT][4];
#pragma unroll
      for (int t = 0; t < SBT; ++t) {
        const uint32_t w = *reinterpret_cast<const uint32_t*>(sm + (16 * t + c) * stride + k + 4 * g);
#pragma unroll
        for (int q = 0; q < 4; ++q) a[t][q] = (float)(int8_t)(w >> (8 * q));
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int u = 0; u < IT; ++u) {
          const float jq = q == 0 ? jv[u].x : q == 1 ? jv[u].y : q == 2 ? jv[u].z : jv[u].w;
#pragma unroll
          for (int t = 0; t < SBT; ++t)
            acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t][q], jq, acc[t][u], 0, 0, 0);
        }
#pragma unroll
      for (int u = 0; u < IT; ++u) jv[u] = jn[u];
    }
    // lane holds F of samples 16 t + 4 g + q at row i0 + 16 u + c
#pragma unroll
    for (int u = 0; u < IT; ++u) {
      const int i = i0 + 16 * u + c;
#pragma unroll
      for (int t = 0; t < SBT; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (i < n) e[t][q] += (double)(acc[t][u][q] * (float)sm[(16 * t + 4 * g + q) * stride + i]);
    }
  }
#pragma unroll
  for (int t = 0; t < SBT; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      double v = e[t][q];
#pragma unroll
      for (int off = 8; off > 0; off >>= 1) v += __shfl_xor(v, off, 16);
      if (c == 0) red[wave][16 * t + 4 * g + q] = v;
    }
  __syncthreads();
  if ((int)threadIdx.x < ns) {
    double tot = 0.0;
    for (int w = 0; w < kDenseWaves; ++w) tot += red[w][threadIdx.x];
    out[b0 + threadIdx.x] = (float)(-0.5 * tot);
  }
}

template <int SBT, int IT>
static void launch_dense_v(int n, int batch, int stride, const float* J, const int8_t* spins, float* out,
                           hipStream_t s) {
  const dim3 grid((batch + 16 * SBT - 1) / (16 * SBT));
  const size_t lds = (size_t)16 * SBT * stride;
  if (n % 4 == 0 && ((uintptr_t)J & 15) == 0)
    hipLaunchKernelGGL((energy_dense_kernel<SBT, IT, true>), grid, dim3(kDenseThreads), lds, s, n, batch, stride, J,
                       spins, out);
  else
    hipLaunchKernelGGL((energy_dense_kernel<SBT, IT, false>), grid, dim3(kDenseThreads), lds, s, n, batch, stride, J,
                       spins, out);
}

static void launch_dense(int n, int batch, const float* J, const int8_t* spins, float* out, hipStream_t s) {
  // rows of spins 16 bytes times an odd number apart: the 16 rows of an A fragment
  // fall on different LDS banks (not at the largest n, where the padding would
  // pass 64 KB)
  int stride = (n + 15) / 16 * 16;
  if (stride / 16 % 2 == 0 && 16 * (stride + 16) <= 65536) stride += 16;
  // rows of J per wave: as many tiles as leave every wave a block; 32 samples per
  // workgroup (each J fragment used twice) where that still gives every compute
  // unit a workgroup and the rows fit 64 KB
  if (n >= 384 && batch >= 4096 && 32 * stride <= 65536) launch_dense_v<2, 4>(n, batch, stride, J, spins, out, s);
  else if (n >= 384) launch_dense_v<1, 4>(n, batch, stride, J, spins, out, s);
  else if (n >= 192) launch_dense_v<1, 2>(n, batch, stride, J, spins, out, s);
  else launch_dense_v<1, 1>(n, batch, stride, J, spins, out, s);
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
