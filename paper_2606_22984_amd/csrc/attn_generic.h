// Band+prefix masked attention for head widths 32 and 64 (the teacher-forced
// pass and its backward), in FP32 arithmetic on the stored Q/K/V.  The 16-wide
// heads take the MFMA kernels of attn_mfma.h; these kernels serve the wider
// heads of the patch-token models (SI, 3D EA settings: two heads at
// d_model 128), whose sequences are short, so their attention is a small part
// of the pass.  Inputs and outputs are those of the MFMA kernels:
//   forward: XM = X + O, LSE (log2 units of the scaled scores);
//   dQ:      DELTA = dO . O, dQ into dQKV and the feature-major copy T;
//   dK/dV:   dK, dV into dQKV and T.
// Thread layout: 4 lanes per row (query or key), each holding DH/4 consecutive
// dims of the head; dot products are summed over the 4 lanes with DPP quad
// permutes.  The other side's rows (keys, or queries for dK/dV) are staged in
// LDS 64 at a time as floats.
#pragma once

#include "attn_mfma.h"

namespace fvan {

constexpr int kGenThreads = 256;
constexpr int kGenRows = kGenThreads / 4;   // queries (keys) per workgroup
constexpr int kGenStage = 64;               // rows of the other side staged at a time

template <int DH>
__host__ __device__ constexpr float gen_inv_sqrt() {
  return DH == 16 ? 0.25f : DH == 32 ? 0.17677669529663688f : 0.125f;
}
template <int DH>
__host__ __device__ constexpr float gen_scale_log2() {
  return gen_inv_sqrt<DH>() * 1.4426950408889634f;
}

// Sum over the 4 lanes of a quad, the same in each of them.
__device__ __forceinline__ float quad_sum(float v) {
  v += dpp<0xB1>(v);
  v += dpp<0x4E>(v);
  return v;
}

// The DH/4 elements of a lane's slice of a row (16-byte aligned), as floats.
template <int Q4, typename T>
__device__ __forceinline__ void load_slice(const T* __restrict__ p, float* out) {
#pragma unroll
  for (int i = 0; i < Q4; i += Chunk<T>::N) {
    Chunk<T> c;
    c.load(p + i);
#pragma unroll
    for (int e = 0; e < Chunk<T>::N; ++e) out[i + e] = c.v[e];
  }
}
template <int Q4>
__device__ __forceinline__ void store_slice(float* __restrict__ p, const float* v) {
#pragma unroll
  for (int i = 0; i < Q4; i += 4) *reinterpret_cast<float4*>(p + i) = make_float4(v[i], v[i + 1], v[i + 2], v[i + 3]);
}

// n rows of DH elements into dst, 16 bytes per load; row(i) is the address of row i.
template <int DH, typename T, typename Row>
__device__ __forceinline__ void stage_rows(float (*dst)[DH + 4], int n, Row&& row) {
  constexpr int VE = Chunk<T>::N, CH = DH / VE;              // elements per load, loads per row
  constexpr int NLD = kGenStage * CH / kGenThreads;
  static_assert(kGenStage * CH % kGenThreads == 0, "whole rounds of loads");
  Chunk<T> c[NLD];
#pragma unroll
  for (int u = 0; u < NLD; ++u) {
    const int idx = threadIdx.x + kGenThreads * u, r = idx / CH;
    c[u].load(row(min(r, n - 1)) + (idx % CH) * VE);
  }
#pragma unroll
  for (int u = 0; u < NLD; ++u) {
    const int idx = threadIdx.x + kGenThreads * u, r = idx / CH;
    if (r < n) store_slice<VE>(&dst[r][(idx % CH) * VE], c[u].v);
  }
}

// The virtual keys (KeyRange order) that a query of the wave's tw0 .. tw0 + 15 sees:
// [0, a1) and [b0, b1).
struct WaveKeys {
  int a1, b0, b1;
  __device__ WaveKeys(const KeyRange& kr, int tw0, int N, int W) {
    const int tw1 = min(tw0 + 15, N - 1);
    a1 = tw0 < N ? min(kr.pend, tw1 + 1) : 0;
    b0 = kr.pend + max(0, tw0 - W - kr.bstart);
    b1 = tw0 < N ? kr.pend + tw1 - kr.bstart + 1 : 0;
  }
};

// ---------------------------------------------------------------- forward
// One workgroup = (64 queries, head, sample).
template <typename KT, int DH>
__global__ __launch_bounds__(kGenThreads) void attn_fwd_gen(const KT* __restrict__ QKV, const float* __restrict__ X,
                                                            float* __restrict__ XM, float* __restrict__ LSE, int N,
                                                            int D, int H, int W, int P) {
  constexpr int Q4 = DH / 4;
  __shared__ __align__(16) float Ks[kGenStage][DH + 4];
  __shared__ __align__(16) float Vs[kGenStage][DH + 4];
  const AttnItem it = attn_item((N + kGenRows - 1) / kGenRows, H);
  const int t0 = it.tile * kGenRows, h = it.h, b = it.b;
  const int t1 = min(t0 + kGenRows, N);
  const int64_t rowbase = (int64_t)b * N;
  const int part = threadIdx.x & 3, tq = t0 + (threadIdx.x >> 2);
  const bool qok = tq < N;
  const int c0 = h * DH + part * Q4;                 // first column of this lane's slice
  float q[Q4], o[Q4];
#pragma unroll
  for (int i = 0; i < Q4; ++i) { q[i] = 0.f; o[i] = 0.f; }
  if (qok) {
    load_slice<Q4>(QKV + (rowbase + tq) * 3 * D + c0, q);
#pragma unroll
    for (int i = 0; i < Q4; ++i) q[i] *= gen_scale_log2<DH>();
  }
  const KeyRange kr(t0, t1, W, P);
  const QueryVis vis(kr, tq, W, qok);
  const WaveKeys wk(kr, t0 + 16 * __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), N, W);
  float mx = -INFINITY, l = 0.f;
  for (int v0 = 0; v0 < kr.nk; v0 += kGenStage) {
    const int nv = min(kGenStage, kr.nk - v0);
    __syncthreads();
    auto krow = [&](int key) { return QKV + (rowbase + kr.pos(v0 + key)) * 3 * D + D + h * DH; };
    stage_rows<DH, KT>(Ks, nv, krow);
    stage_rows<DH, KT>(Vs, nv, [&](int key) { return krow(key) + D; });
    __syncthreads();
    for (int k0 = 0; k0 < nv; k0 += 16) {
      const int vb = v0 + k0;
      if ((vb >= wk.a1) & ((vb + 16 <= wk.b0) | (vb >= wk.b1))) continue;   // no query of the wave sees these keys
      float s[16];
      float mnew = mx;
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int key = k0 + u;
        float d = 0.f;
        if (key < nv) {
#pragma unroll
          for (int i = 0; i < Q4; ++i) d += q[i] * Ks[key][part * Q4 + i];
        }
        d = quad_sum(d);
        s[u] = (key < nv) && vis(v0 + key) ? d : -INFINITY;
        mnew = fmaxf(mnew, s[u]);
      }
      const float corr = mnew == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(mx - mnew);
      l *= corr;
#pragma unroll
      for (int i = 0; i < Q4; ++i) o[i] *= corr;
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        if (s[u] == -INFINITY) continue;
        const float p = __builtin_amdgcn_exp2f(s[u] - mnew);
        l += p;
#pragma unroll
        for (int i = 0; i < Q4; ++i) o[i] += p * Vs[k0 + u][part * Q4 + i];
      }
      mx = mnew;
    }
  }
  if (qok) {
    const int64_t r = rowbase + tq;
    const float inv = 1.0f / l;
    float x[Q4];
    load_slice<Q4>(X + r * D + c0, x);
#pragma unroll
    for (int i = 0; i < Q4; ++i) x[i] = x[i] + o[i] * inv;
    store_slice<Q4>(XM + r * D + c0, x);
    if (part == 0) LSE[r * H + h] = mx + __log2f(l);
  }
}

// ---------------------------------------------------------------- backward: dQ
// One workgroup = (64 queries, head, sample).  O is recovered as XM - X.
template <typename KT, int DH>
__global__ __launch_bounds__(kGenThreads) void attn_bwd_dq_gen(const KT* __restrict__ QKV, const float* __restrict__ X,
                                                               const float* __restrict__ XM,
                                                               const float* __restrict__ dO,
                                                               const float* __restrict__ LSE,
                                                               float* __restrict__ DELTA, float* __restrict__ dQKV,
                                                               float* __restrict__ T, int64_t ldT, int N, int D, int H,
                                                               int W, int P) {
  constexpr int Q4 = DH / 4;
  __shared__ __align__(16) float Ks[kGenStage][DH + 4];
  __shared__ __align__(16) float Vs[kGenStage][DH + 4];
  const AttnItem it = attn_item((N + kGenRows - 1) / kGenRows, H);
  const int t0 = it.tile * kGenRows, h = it.h, b = it.b;
  const int t1 = min(t0 + kGenRows, N);
  const int64_t rowbase = (int64_t)b * N;
  const int part = threadIdx.x & 3, tq = t0 + (threadIdx.x >> 2);
  const bool qok = tq < N;
  const int c0 = h * DH + part * Q4;
  const int64_t r = rowbase + tq;
  float q[Q4], g[Q4], dq[Q4];
  float delta = 0.f, lse = 0.f;
#pragma unroll
  for (int i = 0; i < Q4; ++i) { q[i] = 0.f; g[i] = 0.f; dq[i] = 0.f; }
  if (qok) {
    float xm[Q4], x[Q4];
    load_slice<Q4>(QKV + r * 3 * D + c0, q);
    load_slice<Q4>(dO + r * D + c0, g);
    load_slice<Q4>(XM + r * D + c0, xm);
    load_slice<Q4>(X + r * D + c0, x);
#pragma unroll
    for (int i = 0; i < Q4; ++i) {
      q[i] *= gen_scale_log2<DH>();
      delta += g[i] * (xm[i] - x[i]);
    }
    lse = LSE[r * H + h];
  }
  delta = quad_sum(delta);
  if (qok && part == 0) DELTA[r * H + h] = delta;
  const KeyRange kr(t0, t1, W, P);
  const QueryVis vis(kr, tq, W, qok);
  const WaveKeys wk(kr, t0 + 16 * __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), N, W);
  for (int v0 = 0; v0 < kr.nk; v0 += kGenStage) {
    const int nv = min(kGenStage, kr.nk - v0);
    __syncthreads();
    auto krow = [&](int key) { return QKV + (rowbase + kr.pos(v0 + key)) * 3 * D + D + h * DH; };
    stage_rows<DH, KT>(Ks, nv, krow);
    stage_rows<DH, KT>(Vs, nv, [&](int key) { return krow(key) + D; });
    __syncthreads();
    // the wave's visible keys of this block, in order: [0, a1) then [b0, b1)
    const int na = max(0, min(wk.a1 - v0, nv)), k1 = max(na, wk.b0 - v0), ke = min(wk.b1 - v0, nv);
    for (int it2 = k1 < ke ? na + ke - k1 : na, key = na > 0 ? 0 : k1; it2 > 0; --it2, key = key + 1 == na ? k1 : key + 1) {
      float s = 0.f, dp = 0.f;
#pragma unroll
      for (int i = 0; i < Q4; ++i) {
        s += q[i] * Ks[key][part * Q4 + i];
        dp += g[i] * Vs[key][part * Q4 + i];
      }
      s = quad_sum(s);
      dp = quad_sum(dp);
      const float p = vis(v0 + key) ? __builtin_amdgcn_exp2f(s - lse) : 0.f;
      const float ds = p * (dp - delta);
#pragma unroll
      for (int i = 0; i < Q4; ++i) dq[i] += ds * Ks[key][part * Q4 + i];
    }
  }
  if (qok) {
#pragma unroll
    for (int i = 0; i < Q4; ++i) dq[i] *= gen_inv_sqrt<DH>();
    store_slice<Q4>(dQKV + r * 3 * D + c0, dq);
#pragma unroll
    for (int i = 0; i < Q4; ++i) T[(int64_t)(c0 + i) * ldT + r] = dq[i];
  }
}

// ---------------------------------------------------------------- backward: dK, dV
// One workgroup = (64 keys, head, sample).  The queries that see key j are
// i >= j with i - j <= W, or every i >= j when j < P.
template <typename KT, int DH>
__global__ __launch_bounds__(kGenThreads) void attn_bwd_dkv_gen(const KT* __restrict__ QKV,
                                                                const float* __restrict__ dO,
                                                                const float* __restrict__ LSE,
                                                                const float* __restrict__ DELTA,
                                                                float* __restrict__ dQKV, float* __restrict__ T, int64_t ldT,
                                                                int N, int D, int H, int W, int P) {
  constexpr int Q4 = DH / 4;
  __shared__ __align__(16) float Qs[kGenStage][DH + 4];
  __shared__ __align__(16) float Gs[kGenStage][DH + 4];
  __shared__ float Ls[kGenStage], Ds[kGenStage];
  const AttnItem it = attn_item((N + kGenRows - 1) / kGenRows, H);
  const int j0 = it.tile * kGenRows, h = it.h, b = it.b;
  const int j1 = min(j0 + kGenRows, N);
  const int64_t rowbase = (int64_t)b * N;
  const int part = threadIdx.x & 3, j = j0 + (threadIdx.x >> 2);
  const bool kok = j < N;
  const int c0 = h * DH + part * Q4;
  float k[Q4], v[Q4], dk[Q4], dv[Q4];
#pragma unroll
  for (int i = 0; i < Q4; ++i) { k[i] = 0.f; v[i] = 0.f; dk[i] = 0.f; dv[i] = 0.f; }
  if (kok) {
    load_slice<Q4>(QKV + (rowbase + j) * 3 * D + D + c0, k);
    load_slice<Q4>(QKV + (rowbase + j) * 3 * D + 2 * D + c0, v);
  }
  // queries of the tile's keys: [j0, i_end)
  const int i_end = j0 < P ? N : min(N, j1 - 1 + W + 1);
  // of them, those that see one of the wave's keys jw0 .. jw0 + 15: [jw0, iw_end)
  const int jw0 = j0 + 16 * __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int iw_end = jw0 >= N ? jw0 : (jw0 < P ? i_end : min(i_end, min(N - 1, jw0 + 15) + W + 1));
  for (int i0 = j0; i0 < i_end; i0 += kGenStage) {
    const int nq = min(kGenStage, i_end - i0);
    __syncthreads();
    stage_rows<DH, KT>(Qs, nq, [&](int qi) { return QKV + (rowbase + i0 + qi) * 3 * D + h * DH; });
    stage_rows<DH, float>(Gs, nq, [&](int qi) { return dO + (rowbase + i0 + qi) * D + h * DH; });
    for (int qi = threadIdx.x; qi < nq; qi += kGenThreads) {
      Ls[qi] = LSE[(rowbase + i0 + qi) * H + h];
      Ds[qi] = DELTA[(rowbase + i0 + qi) * H + h];
    }
    __syncthreads();
    for (int qi = max(0, jw0 - i0); qi < min(nq, iw_end - i0); ++qi) {
      float s = 0.f, dp = 0.f;
#pragma unroll
      for (int i = 0; i < Q4; ++i) {
        s += Qs[qi][part * Q4 + i] * k[i];
        dp += Gs[qi][part * Q4 + i] * v[i];
      }
      s = quad_sum(s) * gen_scale_log2<DH>();
      dp = quad_sum(dp);
      const float p = kok && visible(i0 + qi, j, W, P) ? __builtin_amdgcn_exp2f(s - Ls[qi]) : 0.f;
      const float ds = p * (dp - Ds[qi]);
#pragma unroll
      for (int i = 0; i < Q4; ++i) {
        dk[i] += ds * Qs[qi][part * Q4 + i];
        dv[i] += p * Gs[qi][part * Q4 + i];
      }
    }
  }
  if (kok) {
    const int64_t r = rowbase + j;
#pragma unroll
    for (int i = 0; i < Q4; ++i) dk[i] *= gen_inv_sqrt<DH>();
    store_slice<Q4>(dQKV + r * 3 * D + D + c0, dk);
    store_slice<Q4>(dQKV + r * 3 * D + 2 * D + c0, dv);
#pragma unroll
    for (int i = 0; i < Q4; ++i) {
      T[(int64_t)(D + c0 + i) * ldT + r] = dk[i];
      T[(int64_t)(2 * D + c0 + i) * ldT + r] = dv[i];
    }
  }
}

}  // namespace fvan
