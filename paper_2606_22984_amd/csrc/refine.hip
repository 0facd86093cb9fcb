// Local Monte Carlo refinement of sampled configurations (Results, 3D EA;
// Methods, training strategy): checkerboard Metropolis sweeps at inverse
// temperature beta, in place.
//
// The spins live in LDS for all sweeps; a
// sweep updates the sites of colour 0, then those of colour 1, every site's
// local field h_i = sum_j J_ij s_j taken from the configuration at the start
// of the half-sweep (the half-sweep reads one LDS copy of the configuration and
// writes the other).  A flip of s_i changes the
// energy by dE = 2 s_i h_i and is accepted iff u < exp(-beta dE), u from
// Philox4x32-10 with key (seed lo, seed hi), counter (i >> 2, b, sweep, tag),
// word i & 3, u = (word >> 8) 2^-24.  The neighbour table holds every
// neighbour of a site (both directions), -1 for an empty slot.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "device_common.h"
#include "fvan_internal.h"

namespace fvan {

constexpr int kLmcThreads = 256;
constexpr int kLmcMaxSpins = 16384;   // LDS copy of one configuration

// One workgroup per configuration, a thread's sites strided by the workgroup: any
// degree and up to kLmcMaxSpins spins.
__global__ __launch_bounds__(kLmcThreads) void lmc_kernel(const int32_t* __restrict__ nbr, const float* __restrict__ J,
                                                          const int8_t* __restrict__ colour, int n, int degree,
                                                          float beta, int sweeps, uint32_t k0, uint32_t k1,
                                                          uint32_t tag, int8_t* __restrict__ spins,
                                                          int32_t* __restrict__ accepted) {
  // two copies of the configuration: each half-sweep reads buf[p] and writes buf[p ^ 1]
  __shared__ int8_t buf[2][kLmcMaxSpins];
  __shared__ int red[kLmcThreads / 64];
  const int b = blockIdx.x;
  int8_t* row = spins + (int64_t)b * n;
  for (int i = threadIdx.x; i < n; i += kLmcThreads) buf[0][i] = row[i];
  __syncthreads();
  int p = 0, acc = 0;
  for (int k = 0; k < sweeps; ++k) {
    for (int c = 0; c < 2; ++c) {
      for (int i = threadIdx.x; i < n; i += kLmcThreads) {
        int8_t v = buf[p][i];
        if (colour[i] == c) {
          float h = 0.f;
          for (int d = 0; d < degree; ++d) {
            const int j = nbr[(int64_t)i * degree + d];
            if (j >= 0) h += J[(int64_t)i * degree + d] * (float)buf[p][j];
          }
          const float dE = 2.f * (float)v * h;
          const uint4 w = philox4x32_10(make_uint4((uint32_t)(i >> 2), (uint32_t)b, (uint32_t)k, tag), k0, k1);
          const uint32_t x = (i & 3) == 0 ? w.x : (i & 3) == 1 ? w.y : (i & 3) == 2 ? w.z : w.w;
          if (u24(x) < expf(-beta * dE)) {
            v = (int8_t)-v;
            ++acc;
          }
        }
        buf[p ^ 1][i] = v;
      }
      p ^= 1;
      __syncthreads();
    }
  }
  for (int i = threadIdx.x; i < n; i += kLmcThreads) row[i] = buf[p][i];
  if (accepted) {
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
      int t = 0;
      for (int w = 0; w < kLmcThreads / 64; ++w) t += red[w];
      accepted[b] = t;
    }
  }
}

typedef int int32x4 __attribute__((ext_vector_type(4)));
typedef int int32x4u __attribute__((ext_vector_type(4), aligned(4)));   // at any entry of a table

// Entry d of site s of a group's 4 DEG table entries, s = 0 .. 3 (selected, not indexed).
template <int DEG>
__device__ __forceinline__ int of_site(const int32x4 (&t)[DEG], int d, int s) {
  const int e0 = t[d / 4][d % 4], e1 = t[(DEG + d) / 4][(DEG + d) % 4];
  const int e2 = t[(2 * DEG + d) / 4][(2 * DEG + d) % 4], e3 = t[(3 * DEG + d) / 4][(3 * DEG + d) % 4];
  const int lo = s & 1 ? e1 : e0, hi = s & 1 ? e3 : e2;
  return s & 2 ? hi : lo;
}

// The same sweeps with one thread per group of four consecutive sites (the sites
// that share a Philox counter), for degree DEG <= 8 and at most 1024 groups: the
// group's neighbours and bonds stay in registers for all sweeps and its four
// uniforms are drawn once per sweep, where the kernel above reads the table again
// each half-sweep and runs the generator for every site.  A thread holds its sites
// of colour 0 from slot 0 up and the others from slot 3 down, so a half-sweep
// handles two slots (the other two only in a wave where some group is not two and
// two).  lpc threads per configuration (a power of two up to 256, or the whole
// workgroup), blockDim.x / lpc configurations per workgroup.
// The group's entries, 4 DEG in a row in each table, are read 16 bytes at a time and
// given to the slots by selects.  Entry by entry the reads alone took longer than a
// whole sweep of the kernel above, so that refinements of one or two sweeps were
// slower: 16384 configurations of 1000 spins of degree 6, one sweep, 281 us there, 318
// with reads by entry, 88 now; 3000 of 4096 spins 210, 460 and 83.
// Bound by vector issue (the generator, the exponential and the byte reads of the
// neighbours).  The 1000-spin case with 10 sweeps: 2.43 ms with the kernel above, 0.28 now.
template <int DEG>
__global__ __launch_bounds__(1024) void lmc_group_kernel(const int32_t* __restrict__ nbr, const float* __restrict__ J,
                                                         const int8_t* __restrict__ colour, int n, int batch, int lpc,
                                                         float beta, int sweeps, uint32_t k0, uint32_t k1, uint32_t tag,
                                                         int8_t* __restrict__ spins, int32_t* __restrict__ accepted) {
  extern __shared__ uint32_t lds[];          // per configuration: two copies of ngrp words
  __shared__ int count[64];
  const int ngrp = (n + 3) >> 2;
  const int cfg = threadIdx.x / lpc, grp = threadIdx.x % lpc, ncfg = blockDim.x / lpc;
  const int b = blockIdx.x * ncfg + cfg;
  const bool live = grp < ngrp && b < batch;
  uint32_t* mine = lds + (size_t)cfg * 2 * ngrp;
  if (threadIdx.x < 64) count[threadIdx.x] = 0;
  uint32_t cur = 0, order = 0;
  int site[4], col[4];                       // per slot: site of the group, its colour (-1: none)
  int idx[4][DEG];                           // neighbours
  float w[4][DEG];                           // bonds, 0 where there is no neighbour
  int8_t* row = spins + (int64_t)b * n + 4 * grp;
  if (live) {
    int lo = 0, hi = 24;                     // next slot from each end, in bits of `order`
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int i = 4 * grp + e;
      if (i < n) {
        cur |= (uint32_t)(uint8_t)row[e] << (8 * e);
        const int ce = colour[i];
        const int at = ce == 0 ? lo : hi;
        lo += ce == 0 ? 8 : 0;
        hi -= ce == 0 ? 0 : 8;
        order |= (uint32_t)(e | (ce == 0 ? 4 : ce == 1 ? 8 : 12)) << at;
      }
    }
    mine[grp] = cur;
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int o8 = (int)(order >> (8 * u)) & 0xFF;
    site[u] = o8 & 3;
    col[u] = (o8 >> 2) - 1;
  }
  if (live && 4 * grp + 4 <= n) {
    int32x4 t[DEG];
#pragma unroll
    for (int i = 0; i < DEG; ++i) t[i] = reinterpret_cast<const int32x4u*>(nbr)[grp * DEG + i];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int d = 0; d < DEG; ++d) idx[u][d] = of_site<DEG>(t, d, site[u]);
#pragma unroll
    for (int i = 0; i < DEG; ++i) t[i] = reinterpret_cast<const int32x4u*>(J)[grp * DEG + i];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int d = 0; d < DEG; ++d) {
        const bool ok = idx[u][d] >= 0 && idx[u][d] < n;
        w[u][d] = ok ? __int_as_float(of_site<DEG>(t, d, site[u])) : 0.f;
        idx[u][d] = ok ? idx[u][d] : 0;
      }
  } else {
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int d = 0; d < DEG; ++d) {
        const int64_t o = (int64_t)(4 * grp + site[u]) * DEG + d;
        const int j = live && col[u] >= 0 ? nbr[o] : -1;
        const bool ok = j >= 0 && j < n;
        idx[u][d] = ok ? j : 0;
        w[u][d] = ok ? J[o] : 0.f;
      }
  }
  const bool more0 = __any(col[2] == 0 || col[3] == 0), more1 = __any(col[0] == 1 || col[1] == 1);
  __syncthreads();
  int p = 0, acc = 0;
  for (int k = 0; k < sweeps; ++k) {
    const uint4 x = philox4x32_10(make_uint4((uint32_t)grp, (uint32_t)b, (uint32_t)k, tag), k0, k1);
    // the two words of each half as one value, so that a site's word is a shift away
    const uint64_t x01 = (uint64_t)x.y << 32 | x.x, x23 = (uint64_t)x.w << 32 | x.z;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int8_t* from = reinterpret_cast<const int8_t*>(mine + p * ngrp);
      uint32_t next = cur;
      auto flip = [&](auto slot) {
        constexpr int u = decltype(slot)::value;
        float h = 0.f;
#pragma unroll
        for (int d = 0; d < DEG; ++d) h += w[u][d] * (float)from[idx[u][d]];
        const int sh = 8 * site[u];
        const int8_t v = (int8_t)(cur >> sh);
        const float dE = 2.f * (float)v * h;
        const uint32_t r = (uint32_t)((site[u] & 2 ? x23 : x01) >> (32 * (site[u] & 1)));
        if (col[u] == c && u24(r) < expf(-beta * dE)) {
          next = (next & ~(0xFFu << sh)) | ((uint32_t)(uint8_t)(int8_t)-v << sh);
          ++acc;
        }
      };
      if (c == 0 || more1) {
        flip(std::integral_constant<int, 0>());
        flip(std::integral_constant<int, 1>());
      }
      if (c == 1 || more0) {
        flip(std::integral_constant<int, 2>());
        flip(std::integral_constant<int, 3>());
      }
      cur = next;
      p ^= 1;
      if (live) mine[p * ngrp + grp] = cur;
      __syncthreads();
    }
  }
  if (live) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (4 * grp + e < n) row[e] = (int8_t)(cur >> (8 * e));
    if (accepted && acc) atomicAdd(&count[cfg], acc);
  }
  __syncthreads();
  if (accepted && grp == 0 && b < batch) accepted[b] = count[cfg];
}

hipError_t launch_lmc(int32_t n, int32_t degree, const int32_t* nbr, const float* J, const int8_t* colour,
                      int32_t batch, double beta, int32_t sweeps, uint64_t seed, uint32_t stream_tag, int8_t* spins,
                      int32_t* accepted, hipStream_t s) {
  if (n < 1 || n > kLmcMaxSpins || batch < 1) return hipErrorInvalidValue;
  const uint32_t k0 = (uint32_t)(seed & 0xFFFFFFFFu), k1 = (uint32_t)(seed >> 32);
  // one thread per group of four sites where the groups of a configuration fit one
  // workgroup and a group's neighbours fit registers (2D lattices: 4, 3D: 6)
  const int ngrp = (n + 3) / 4;
  if (ngrp <= 1024 && degree <= 8) {
    int lpc = 4;                             // threads per configuration
    while (lpc < ngrp && lpc < 256) lpc *= 2;
    if (lpc < ngrp) lpc = (ngrp + 63) / 64 * 64;
    const int threads = std::max(lpc, 256), ncfg = threads / lpc;
    const dim3 grid((batch + ncfg - 1) / ncfg), block(threads);
    const size_t bytes = (size_t)ncfg * 2 * ngrp * 4;
    decltype(&lmc_group_kernel<1>) kernels[8] = {lmc_group_kernel<1>, lmc_group_kernel<2>, lmc_group_kernel<3>,
                                                 lmc_group_kernel<4>, lmc_group_kernel<5>, lmc_group_kernel<6>,
                                                 lmc_group_kernel<7>, lmc_group_kernel<8>};
    hipLaunchKernelGGL(kernels[degree - 1], grid, block, bytes, s, nbr, J, colour, n, batch, lpc, (float)beta, sweeps,
                       k0, k1, stream_tag, spins, accepted);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(lmc_kernel, dim3(batch), dim3(kLmcThreads), 0, s, nbr, J, colour, n, degree, (float)beta, sweeps,
                     k0, k1, stream_tag, spins, accepted);
  return hipGetLastError();
}

}  // namespace fvan
