// Overlap distribution (Eq. overlap_distribution) of a batch of independent
// samples: counts[k] = number of pairs a < b whose configurations agree on k
// sites, i.e. whose overlap q = (1/N) s_a . s_b equals 2k/N - 1.
//
// The pair products are the dense contraction Q = S S^T of the +-1 spins, done
// on int8 MFMA (16x16x64, int32 accumulation: exact).  A workgroup takes BT x BT
// blocks (I <= J) of Q from a grid-stride list of the upper triangle.  Both
// blocks' rows are staged in LDS 64 spins at a time, in two alternating buffers
// (the next step's rows are fetched into registers during the current products),
// and a wave owns BT/WR x BT/WC of the block.  Each pair a < b adds one count to
// an LDS histogram, which the workgroup adds to the global counts once at the end
// (integer atomics: the result does not depend on their order).
//
// Overlaps concentrate on few bins, so the histogram is kept in up to 16 copies,
// interleaved so that the lanes of a 16-lane row never meet on an address; one
// copy per bin made the LDS atomics the bound.  With 64 x 64 blocks read straight
// from L2 by every wave and one copy, 16384 samples of 1000 spins took 936 us; now
// 249 us (1.08e15 int8 operations/s), the atomics about half of it.
#include <algorithm>
#include <cmath>

#include "device_common.h"
#include "fvan_internal.h"

namespace fvan {

constexpr int kOvMaxSpins = 16000;
constexpr int kOvHistBytes = 65536;      // LDS of the histogram copies, 256 x 256 blocks
constexpr int kOvHistSmall = 8192;       // and smaller blocks
constexpr int kOvPitch = 80;             // bytes per staged row: 64 spins + padding (conflict-free 16-byte reads)

typedef int int4v __attribute__((ext_vector_type(4)));

// 16 spins of a row starting at k, zero past n (any alignment)
__device__ __forceinline__ uint4 load16(const int8_t* __restrict__ row, int k, int n) {
  uint4 v = make_uint4(0u, 0u, 0u, 0u);
  if (k + 16 <= n) {
    __builtin_memcpy(&v, row + k, 16);
  } else if (k < n) {
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < 16; ++j) w[j >> 2] |= (k + j < n ? (uint32_t)(uint8_t)row[k + j] : 0u) << (8 * (j & 3));
    v = make_uint4(w[0], w[1], w[2], w[3]);
  }
  return v;
}

template <int BT, int WR, int WC>
__global__ __launch_bounds__(64 * WR * WC) void overlap_kernel(const int8_t* __restrict__ S, int B, int n, int copies,
                                                               unsigned long long* __restrict__ counts) {
  constexpr int T = 64 * WR * WC;                    // threads
  constexpr int RT = BT / WR / 16, CT = BT / WC / 16;   // 16-row and 16-column tiles of a wave
  constexpr int NP = 2 * BT * 4 / T;                 // 16-byte pieces a thread stages per step
  static_assert(2 * BT * 4 % T == 0, "whole pieces per thread");
  __shared__ __align__(16) int8_t rows[2][2 * BT][kOvPitch];   // block I's rows, then block J's
  extern __shared__ unsigned int hist[];             // [n + 2][copies]; bin n + 1 takes what is not counted
  for (int k = threadIdx.x; k < (n + 1) * copies; k += T) hist[k] = 0u;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r = lane & 15, g = lane >> 4;
  const int wr = wave / WC, wc = wave % WC, copy = lane & (copies - 1);
  const int cb = __builtin_ctz(copies);
  const unsigned most = 2u * n + 2u, low = copies - 1u;
  const int nblk = (B + BT - 1) / BT;
  const int npairs = nblk * (nblk + 1) / 2;
  const int steps = (n + 63) / 64;
  for (int p = blockIdx.x; p < npairs; p += gridDim.x) {
    // p-th block pair (I, J), I <= J, in row-major upper-triangle order
    int I = (int)floor(((2.0 * nblk + 1.0) - sqrt((2.0 * nblk + 1.0) * (2.0 * nblk + 1.0) - 8.0 * p)) * 0.5);
    while (I > 0 && I * (2 * nblk - I + 1) / 2 > p) --I;
    while ((I + 1) * (2 * nblk - I) / 2 <= p) ++I;
    const int J = I + (p - I * (2 * nblk - I + 1) / 2);
    uint4 pre[NP];
    auto fetch = [&](int k) {
#pragma unroll
      for (int u = 0; u < NP; ++u) {
        const int x = threadIdx.x + T * u, row = x >> 2;
        const int s = (row < BT ? I * BT + row : J * BT + row - BT);
        pre[u] = load16(S + (int64_t)min(s, B - 1) * n, k + 16 * (x & 3), n);
      }
    };
    auto commit = [&](int buf) {
#pragma unroll
      for (int u = 0; u < NP; ++u) {
        const int x = threadIdx.x + T * u;
        *reinterpret_cast<uint4*>(&rows[buf][x >> 2][16 * (x & 3)]) = pre[u];
      }
    };
    int4v acc[RT][CT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < CT; ++j) acc[i][j] = int4v{n, n, n, n};   // Q + n, twice the bin
    fetch(0);
    commit(0);
    __syncthreads();                                 // also: the histogram is cleared
    for (int st = 0; st < steps; ++st) {
      if (st + 1 < steps) fetch(64 * (st + 1));
      int4v fa[RT];
#pragma unroll
      for (int i = 0; i < RT; ++i)
        fa[i] = *reinterpret_cast<const int4v*>(&rows[st & 1][(wr * RT + i) * 16 + r][16 * g]);
#pragma unroll
      for (int j = 0; j < CT; ++j) {
        const int4v fb = *reinterpret_cast<const int4v*>(&rows[st & 1][BT + (wc * CT + j) * 16 + r][16 * g]);
#pragma unroll
        for (int i = 0; i < RT; ++i) acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[i], fb, acc[i][j], 0, 0, 0);
      }
      if (st + 1 < steps) commit((st + 1) & 1);      // last read in step st - 1
      __syncthreads();
    }
    // lane holds Q + n of (row 16 i + 4 g + q of the wave's rows, row 16 j + r of its
    // columns): bin (Q + n) >> 1, in [0, n] for +-1 spins (other values go to bin n + 1)
    const bool inside = I < J && (J + 1) * BT <= B;  // every pair of the block counts
    auto slot = [&](int v) {
      const unsigned m = min((unsigned)v, most);
      return (((cb ? m << (cb - 1) : m >> 1)) & ~low) | (unsigned)copy;
    };
    if (inside) {
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) atomicAdd(&hist[slot(acc[i][j][q])], 1u);
    } else {
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int ra = I * BT + (wr * RT + i) * 16 + 4 * g + q, rb = J * BT + (wc * CT + j) * 16 + r;
            if (ra < rb && rb < B) atomicAdd(&hist[slot(acc[i][j][q])], 1u);
          }
    }
  }
  __syncthreads();
  for (int k = threadIdx.x; k <= n; k += T) {
    unsigned long long c = 0;
    for (int u = 0; u < copies; ++u) c += hist[k * copies + ((u + k) & (copies - 1))];
    if (c) atomicAdd(&counts[k], c);
  }
}

__global__ void zero_u64_kernel(unsigned long long* p, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0ull;
}

hipError_t launch_overlap(int32_t batch, int32_t n, const int8_t* spins, unsigned long long* counts, hipStream_t s) {
  if (batch < 1 || n < 1 || n > kOvMaxSpins) return hipErrorInvalidValue;
  hipLaunchKernelGGL(zero_u64_kernel, dim3((n + 256) / 256), dim3(256), 0, s, counts, n + 1);
  const auto pairs = [&](int bt) {
    const int64_t b = (batch + bt - 1) / bt;
    return b * (b + 1) / 2;
  };
  // as many histogram copies as fit `bytes`
  const auto launch = [&](auto kern, int threads, int64_t grid, size_t bytes) {
    int copies = 16;
    while (copies > 1 && (size_t)(n + 2) * copies * 4 > bytes) copies /= 2;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(threads), (size_t)(n + 2) * copies * 4, s, spins, batch, n,
                       copies, counts);
  };
  // Block size by the rounds of workgroups over 256 compute units.  A block pair of 64
  // costs the most reads per product but the least on a chip that it does not fill: up
  // to one per unit, or two while their histograms leave room for two (1800 samples of
  // 12000 spins: 111 us, with 128 153; of 16000, where one fits: 229 with 64, 166 with
  // 128).  Two workgroups of 128 share a unit, and a round of theirs takes 2/3 of a round
  // of one of 256 (5000 samples of 1000 spins, 2 against 1 rounds: 45 and 34 us; 3000, 1
  // and 1: 24 and 31; 6000, 3 and 2: 62 and 60, and of 64 spins 17 and 19).
  // The smaller blocks get 8 KB of histogram copies: with 64 KB one workgroup had a unit
  // to itself (2000 samples of 1000 spins: 42 us with 64 and 64 KB, 25 with 64 and 8 KB, 20
  // with 128; the kernel before the staged blocks took 29).
  const int64_t p64 = pairs(64), p128 = pairs(128), p256 = pairs(256);
  const int64_t r128 = (p128 + 511) / 512, r256 = (p256 + 255) / 256;
  if (p64 <= 256 || (p64 <= 450 && n <= 14000))
    launch(overlap_kernel<64, 2, 2>, 256, p64, kOvHistSmall);
  else if (2 * r128 <= 3 * r256)
    launch(overlap_kernel<128, 2, 2>, 256, std::min<int64_t>(p128, 512), kOvHistSmall);
  else
    launch(overlap_kernel<256, 4, 2>, 512, std::min<int64_t>(p256, 256), kOvHistBytes);
  return hipGetLastError();
}

}  // namespace fvan
