// KV-cached ancestral sampling (Alg. 2 of the paper) for gfx950.
//
// One workgroup (8 waves) owns a tile of up to KM = 32 (or 16) samples and runs every
// step t = 0..N-1 and every layer without leaving the kernel: samples are
// independent, so no grid-wide synchronisation is ever needed.  Per layer step:
//   LN1 (16 lanes per sample, DPP reductions)
//   QKV = LN1(h) W^T + b on MFMA (KM samples x 3d: every weight fragment a wave
//        loads feeds both 16-sample row tiles, which halves the weight traffic
//        per sample); q_t, k_t, v_t go to LDS
//   attention: one wave per sample, K/V rows streamed with 16-byte coalesced
//        loads (the step's own row taken from LDS and appended to the sample's
//        cache slot), per-head dot products and an online softmax reduced with
//        lane swaps; the heads' concatenation is added to h (no W_O)
//   LN2 + FFN (4d hidden kept in LDS) on MFMA, residual added in place
// then the head, the Philox draw and the decision.  The KV cache of a sample
// and layer holds the prefix positions [0, P) and a ring of the last R band
// positions, so the visible keys of step t are always slots [0, nvis).
//
// What bounds a layer step (2D L=16 model, 16 samples per workgroup, 23100 clocks
// before): the attention's vector instructions (about 5600 clocks of issue per SIMD,
// and a latency of memory before them), then an L2 latency at the head of each of
// the other phases.  So the loads are issued a phase ahead (below), the merge of the
// attention's row groups keeps only the elements a lane will add, and a layer's
// offsets are compile-time constants (20 fewer scalar registers to spill).
// 10.24 -> 8.56 ms per 4096 samples, N=16 SK 211 -> 141 us per 1024 with the tile rule
// (sample_tile); 2D groups 45.1 -> 36.9 ms; same samples bit for bit.
//
// Template parameters: D = d_model, MODE = precision, DH = head width (16, 32
// or 64), WIDE = caches past 32-bit offsets (below), TOK = a model over 2^D-spin patch tokens: the head has `vocab`
// outputs, the token is drawn from the V-way softmax by one uniform (walking
// the vocabulary from the top, so V = 2 is the binary rule) and fed to the token
// embedding of the next position; the token, not a spin, is written out.
//
// The kernel templates are instantiated in decode.hip (the single-spin kernels
// with 16-wide heads) and decode_ext.hip (other head widths and token models).
#pragma once

#include <type_traits>

#include "device_common.h"
#include "fvan_model.h"

namespace fvan {

typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kMaxVocab = 256;

// KM: samples per workgroup, 32 (two 16-row MFMA tiles: every weight fragment
// feeds both) or 16 (one tile; twice the workgroups for a batch).
template <int D, int MODE, bool TOK, int KM>
struct DecodeSmem {
  typedef typename Mode<MODE>::ActT A;
  static constexpr int PAD = 16 / (int)sizeof(A);
  static constexpr int LDA = D + PAD;
  static constexpr int LDH = 4 * D + PAD;
  static constexpr int LDZ = kMaxVocab + 1;
  __align__(16) float h[KM][D];
  A a[KM][LDA];
  union {
    float q[KM][D];
    A hid[KM][LDH];
    float z[TOK ? KM : 1][TOK ? LDZ : 1];   // logits of the vocab-way head
  } u;
  // k_t and v_t of the tile's samples for the layer in progress
  __align__(16) typename Mode<MODE>::KvT kv[KM][2][D];
  int tok[KM];
  int8_t sbuf[KM][64];
  // FFN2 partial sums of the waves that take the upper K ranges in split mode
  // when d < 128 (fewer output tiles than waves; FP32 mode measured no gain)
  static constexpr int KP = Mode<MODE>::SPLIT && D / 16 < kWaves ? kWaves / (D / 16) - 1 : 0;
  float kpart[KP > 0 ? KP : 1][KP > 0 ? KM : 1][KP > 0 ? D : 1];
};


__device__ __forceinline__ float reduce16(float v) { return row_sum16(v); }

// The K/V block of one sample and layer as a raw buffer: a lane with nothing to load
// or store gives an offset past the end (loads return zero, stores are dropped), so
// no branch surrounds the access and the compiler knows how many loads are in flight
// behind the one it waits for.  Loads are non-temporal, so that the stream does not
// push the layer weights out of L2.
// The block must fit 32-bit offsets (decode_wide).  The WIDE form of the kernel takes
// a buffer per batch and plane from its 64-bit address instead, any length of cache; its
// scalar registers are why it is not the only form (N=16 SK, 1024 samples: 150 against
// 140 us; 2D L=16: 9.49 against 8.55 ms; a branch between the two: 166 us and 9.42 ms).
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
typedef __amdgpu_buffer_rsrc_t kv_rsrc_t;
constexpr int kNoLane = 0x7FFFFFF0;          // past the end of any block
__device__ __forceinline__ kv_rsrc_t kv_rsrc(void* base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00020000);
}
__device__ __forceinline__ uint4 kv_load16(kv_rsrc_t r, int voff, int soff) {
  const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 2);
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void kv_store16(kv_rsrc_t r, const uint4& x, int voff) {
  const u32x4_t v = {x.x, x.y, x.z, x.w};
  __builtin_amdgcn_raw_buffer_store_b128(v, r, voff, 0, 0);
}

// (a, b) of a lane and of lane ^ off become (the a of the pair's lower lane, the a of
// its upper lane) in the lower lane and the same of b in the upper one: each lane of
// the pair ends up with both lanes' values of one of the two.  off = 4, 8, 16 or 32.
__device__ __forceinline__ void lane_pair(float& a, float& b, int off) {
  const uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
  if (off == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(ua, ub, false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
  } else if (off == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(ua, ub, false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
  } else if (off == 8) {                     // row_ror:8 into the upper (lower) half of each row only
    a = __int_as_float(__builtin_amdgcn_update_dpp((int)ua, (int)ub, 0x128, 0xF, 0xC, false));
    b = __int_as_float(__builtin_amdgcn_update_dpp((int)ub, (int)ua, 0x128, 0xF, 0x3, false));
  } else {
    const bool up = threadIdx.x & off;
    const float x = __shfl_xor(up ? a : b, off);
    const float keep = up ? b : a;
    a = up ? x : keep;
    b = up ? keep : x;
  }
}

// x, hidden from loop-invariant code motion: what is computed from it stays where it
// is used (hoisted out of the step and layer loops, the lane's many addresses took
// the registers of the loads in flight and spilled)
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// LayerNorm of the KM residual rows into the MFMA operand buffer (16 lanes per row).
// In split mode the output is written already split, once: each group of 8
// consecutive elements of a row is a BF16 hi uint4 followed by its lo uint4 (the
// same hi/lo as the GEMMs' own split of FP32 operands), so the QKV and FFN1
// products read their A fragments without converting them per output tile.
// The lane's gains and shifts are loaded ahead (LnParams).
template <int D, int MODE>
struct LnParams {
  static constexpr int PER = D / 16;
  float g[PER], b[PER];
  __device__ __forceinline__ void load(const float* __restrict__ pg, const float* __restrict__ pb) {
    const int part = opaque(threadIdx.x & 15);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int k = Mode<MODE>::SPLIT ? part * PER + i : part + 16 * i;
      g[i] = pg[k];
      b[i] = pb[k];
    }
  }
};
template <int D, int MODE, bool TOK, int KM>
__device__ __forceinline__ void ln_rows(DecodeSmem<D, MODE, TOK, KM>& sm, const LnParams<D, MODE>& lp) {
  typedef typename Mode<MODE>::ActT T;
  constexpr int PER = D / 16;
  constexpr bool SPLIT = Mode<MODE>::SPLIT;
  const int tid = opaque(threadIdx.x), m = tid >> 4, part = tid & 15;
  if (m >= KM) return;
  float x[PER];
  float s = 0.f;
  // split mode: PER consecutive elements per lane; otherwise strided by 16
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    x[i] = sm.h[m][SPLIT ? part * PER + i : part + 16 * i];
    s += x[i];
  }
  const float mean = reduce16(s) * (1.0f / D);
  float v = 0.f;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    x[i] -= mean;
    v += x[i] * x[i];
  }
  const float rstd = rsqrtf(reduce16(v) * (1.0f / D) + kLnEps);
  if constexpr (SPLIT) {
    static_assert(PER % 2 == 0 && 8 % PER == 0, "a lane's elements lie in one 8-element group");
    float y[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) y[i] = x[i] * rstd * lp.g[i] + lp.b[i];
    // hi = bf16(y), lo = bf16(y - hi), two elements per 32-bit word
    uint32_t hw[PER / 2], lw[PER / 2];
#pragma unroll
    for (int i = 0; i < PER; i += 2) {
      const f32x2_t v2 = {y[i], y[i + 1]};
      const bf16x2_t h2 = __builtin_convertvector(v2, bf16x2_t);
      uint32_t hb;
      __builtin_memcpy(&hb, &h2, 4);
      const f32x2_t r2 = {y[i] - __uint_as_float(hb << 16), y[i + 1] - __uint_as_float(hb & 0xFFFF0000u)};
      const bf16x2_t l2 = __builtin_convertvector(r2, bf16x2_t);
      hw[i / 2] = hb;
      __builtin_memcpy(&lw[i / 2], &l2, 4);
    }
    uint32_t* row = reinterpret_cast<uint32_t*>(&sm.a[m][0]);
    const int j = part * PER / 8, o = (part * PER % 8) / 2;   // group, 32-bit word inside the group's uint4
#pragma unroll
    for (int w = 0; w < PER / 2; ++w) {
      row[8 * j + o + w] = hw[w];
      row[8 * j + 4 + o + w] = lw[w];
    }
  } else {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int k = part + 16 * i;
      sm.a[m][k] = from_f<T>(x[i] * rstd * lp.g[i] + lp.b[i]);
    }
  }
}

// The output tiles nt = nt0, nt0 + step, ... < ntn of A[16 NRT x K] (LDS, row
// stride lda) . pack, each finished tile handed to epi(nt, acc0, acc1).  The
// weight fragments come G chunks per round, and the loads of the next two rounds
// (of this tile or of the wave's next one) are in flight while a round multiplies.
// begin() issues the first two rounds: it is called a phase ahead, so that their L2
// latency passes under that phase (the weights do not depend on it); loaded(), once
// every load of the product has been issued, is where the caller begins the next
// phase's loads (a wave's loads return in order, so nothing a phase waits for is
// issued behind a longer load).  Per tile the chunks are summed in order, as a
// single pass over the tile would; acc1 stays zero when NRT = 1.
// PRE: A holds split-mode operands written by ln_rows (per 8-element group a hi
// uint4, then its lo uint4; row stride lda elements of Mode<2>::ActT).
// LO: hi-to-lo distance of a split pack, in fragments.
template <int MODE, int K, int LO>
struct TileLoads {
  static constexpr int KC = Mode<MODE>::KC;
  static constexpr int NC = K / KC;
  static constexpr int GM = Mode<MODE>::SPLIT ? 2 : 4;
  static constexpr int G = NC < GM ? NC : GM;
  static constexpr int R = NC / G;          // rounds per tile
  static_assert(NC % G == 0, "K chunks in groups of G");
  uint4 h0[G], l0[G], h1[G], l1[G];         // the first two rounds
  const uint4* pack;
  __device__ __forceinline__ void load(int t, int rr, int lane, uint4* h, uint4* l) const {
#pragma unroll
    for (int u = 0; u < G; ++u) {
      const uint4* bp = pack + (uint32_t)((t * NC + rr * G + u) * 64 + lane);
      h[u] = bp[0];
      l[u] = Mode<MODE>::SPLIT ? bp[LO] : h[u];
    }
  }
  // tile and round after (t, rr)
  static __device__ __forceinline__ void advance(int& t, int& rr, int step) {
    if (++rr == R) {
      rr = 0;
      t += step;
    }
  }
  // (a wave with fewer rounds loads its last tile's again: without branches the
  // registers are free from one use to the next load)
  __device__ __forceinline__ void begin(const uint4* __restrict__ p, int nt0, int ntn, int step, int lane) {
    pack = p;
    load(min(nt0, ntn - 1), 0, lane, h0, l0);
    int t = nt0, r = 0;
    advance(t, r, step);
    load(min(t, ntn - 1), r, lane, h1, l1);
  }
};

// MAXT: the most tiles a wave has.
template <int MODE, int K, int NRT, bool PRE, int MAXT, int LO, typename Epi, typename Loaded>
__device__ __forceinline__ void mfma_tiles(TileLoads<MODE, K, LO>& w, const typename Mode<MODE>::ActT* A, int lda, int nt0,
                                           int ntn, int step, int lane, Epi&& epi, Loaded&& loaded) {
  typedef TileLoads<MODE, K, LO> W;
  constexpr int KC = W::KC, G = W::G, R = W::R;
  if (nt0 >= ntn) {
    loaded();
    return;
  }
  static_assert(!PRE || Mode<MODE>::SPLIT, "pre-split operands in split mode only");
  const typename Mode<MODE>::ActT* arow = A + (lane & 15) * lda + (lane >> 4) * (KC / 4);
  const typename Mode<MODE>::ActT* arow1 = arow + 16 * lda;
  // pre-split: lane (g, c) takes group 4 kc + g of row c: uint4s 2 (4 kc + g) and + 1
  const uint4* prow = reinterpret_cast<const uint4*>(A) + (lane & 15) * (lda * (int)sizeof(*A) / 16) + 2 * (lane >> 4);
  const uint4* prow1 = prow + 16 * (lda * (int)sizeof(*A) / 16);
  floatx4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = acc0;
  auto multiply = [&](int nt, int r, const uint4* bh, const uint4* bl) FVAN_INLINE {
#pragma unroll
    for (int u = 0; u < G; ++u) {
      const int kc = r * G + u;
      if constexpr (PRE) {
        // the same three products in the same order as Frag<2>::step1v / step2v
        static_assert(KC == 32, "four 8-element groups per K chunk");
        const uint4 xh = prow[8 * kc], xl = prow[8 * kc + 1];
        if constexpr (NRT == 2) {
          const uint4 yh = prow1[8 * kc], yl = prow1[8 * kc + 1];
          acc0 = mfma_bf16(xl, bh[u], acc0);
          acc1 = mfma_bf16(yl, bh[u], acc1);
          acc0 = mfma_bf16(xh, bl[u], acc0);
          acc1 = mfma_bf16(yh, bl[u], acc1);
          acc0 = mfma_bf16(xh, bh[u], acc0);
          acc1 = mfma_bf16(yh, bh[u], acc1);
        } else {
          acc0 = mfma_bf16(xl, bh[u], acc0);
          acc0 = mfma_bf16(xh, bl[u], acc0);
          acc0 = mfma_bf16(xh, bh[u], acc0);
        }
      } else {
        const int k = kc * KC;
        if constexpr (NRT == 2)
          Frag<MODE>::step2v(arow + k, arow1 + k, bh[u], bl[u], acc0, acc1);
        else
          Frag<MODE>::step1v(arow + k, bh[u], bl[u], acc0);
      }
    }
    if (r == R - 1) {
      epi(nt, acc0, acc1);
      acc0 = floatx4{0.f, 0.f, 0.f, 0.f};
      acc1 = acc0;
    }
  };
  int nt = nt0, r = 0, nt1 = nt0, r1 = 0;
  W::advance(nt1, r1, step);
  if constexpr (MAXT * R > 2) {
    int nt2 = nt1, r2 = r1;
    W::advance(nt2, r2, step);
    while (nt2 < ntn) {                     // a round beyond the two in flight
      uint4 mh[G], ml[G];
      w.load(nt2, r2, lane, mh, ml);
      multiply(nt, r, w.h0, w.l0);
#pragma unroll
      for (int u = 0; u < G; ++u) {
        w.h0[u] = w.h1[u];
        w.l0[u] = w.l1[u];
        w.h1[u] = mh[u];
        w.l1[u] = ml[u];
      }
      nt = nt1;
      r = r1;
      nt1 = nt2;
      r1 = r2;
      W::advance(nt2, r2, step);
    }
  }
  loaded();
  multiply(nt, r, w.h0, w.l0);
  if (nt1 < ntn) multiply(nt1, r1, w.h1, w.l1);
}

// bias[i] of the wave's i-th output tile, chosen without indexing registers
template <int T>
__device__ __forceinline__ float pick(const float (&v)[T], int i) {
  float x = v[0];
#pragma unroll
  for (int k = 1; k < T; ++k) x = i == k ? v[k] : x;
  return x;
}

template <int D, int MODE, int DH, bool TOK, int KM, bool WIDE>
__device__ void decode_tile(DecodeSmem<D, MODE, TOK, KM>& sm, const DecodeUnit& U, int local_tile) {
  typedef typename Mode<MODE>::KvT T;
  typedef DecodeSmem<D, MODE, TOK, KM> Sm;
  constexpr int NRT = KM / 16;          // 16-row MFMA tiles
  static_assert(KM == 16 || KM == 32, "16 or 32 samples per workgroup");
  constexpr int VEC = Chunk<T>::N;
  constexpr int LPR = D / VEC;          // lanes per K/V row
  constexpr int RPL = 64 / LPR;         // rows per wave load
  constexpr int LPH = DH / VEC;         // lanes per head
  // rows per lane in flight: 5 at d = 64 (40-row batches: a 2D lattice step's
  // visible keys, up to 2L + 2, take one or two batches instead of two or three;
  // measured 11% faster at L = 16), 4 otherwise (at d = 128 a fifth row spills
  // registers and gains nothing)
  constexpr int UNR = D == 64 ? 5 : 4;
  static_assert(DH == 16 || DH == 32 || DH == 64, "head width 16, 32 or 64");
  static_assert(LPH >= 2 && LPH <= LPR, "a head spans 2 .. LPR lanes of a row");
  // 1/sqrt(DH) * log2(e)
  constexpr float kScaleLog2 = (DH == 16 ? 0.25f : DH == 32 ? 0.17677669529663688f : 0.125f) * 1.4426950408889634f;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b0 = local_tile * U.tile;   // U.tile <= KM samples per workgroup
  const int nb = min(U.tile, U.B - b0);
  const int N = U.N, P = U.P, R = U.R, S = U.S, nl = U.n_layers, dt = U.d_token;
  const float* __restrict__ theta = U.theta;
  const char* wbase = reinterpret_cast<const char*>(U.wpack);
  T* kvbase = reinterpret_cast<T*>(U.kv);
  const size_t plane = (size_t)S * D;   // elements of one K (or V) block

  // head-phase ownership: thread 16*m handles sample row m
  const int hm = tid >> 4, hpart = tid & 15;
  float lq = 0.f;
  float ur[4] = {0.f, 0.f, 0.f, 0.f};
  if (tid < KM) sm.tok[tid] = 0;   // start token

  // Loads that do not depend on the step's arithmetic are issued ahead of the phase
  // that uses them: the layer's small parameters and first weight rounds a phase
  // ahead, the K/V rows of the layer's first batch from the previous layer's FFN2.
  // Exposed, each phase began with an L2 latency and the attention with a memory
  // latency.  (The second batch from there as well: 9.26 against 8.58 ms for the 2D
  // L=16 sampling, as a compute unit's loads all in one phase wait for its 64 bytes
  // per clock of L1.)
  constexpr int TQ = (3 * D / 16 + kWaves - 1) / kWaves;   // output tiles per wave: QKV, FFN1
  constexpr int T1 = (4 * D / 16 + kWaves - 1) / kWaves;
  constexpr int NT2 = D / 16;                              // FFN2 output tiles
  constexpr int SK = Sm::KP + 1;                           // waves per FFN2 output tile (K ranges)
  constexpr int NCS = 4 * D / Mode<MODE>::KC / SK;         // K chunks per range
  constexpr int LOQ = 3 * D * D / 8, LOF = 4 * D * D / 8;
  const int tile2 = SK > 1 ? wave % NT2 : wave, part2 = SK > 1 ? wave / NT2 : 0;
  TileLoads<MODE, D, LOQ> wq;
  TileLoads<MODE, D, LOF> w1;
  TileLoads<MODE, 4 * D / SK, LOF> w2;
  LnParams<D, MODE> ln1, ln2;
  float bq[TQ], b1[T1], b2;
  constexpr LayerOffsets LO = layer_offsets(D);
  const float* __restrict__ theta0 = theta + U.layer0;
  auto layer_theta = [&](int l) FVAN_INLINE { return theta0 + (uint32_t)(l * (int)LO.stride); };
  auto layer_pack = [&](int l, int64_t off) FVAN_INLINE {
    return reinterpret_cast<const uint4*>(wbase + (uint32_t)(l * (int)pack_layer_bytes(D) + (int)off));
  };
  auto begin_qkv = [&](int l) FVAN_INLINE {
    const int lane = opaque(tid & 63);
    const float* lp = layer_theta(l);
    ln1.load(lp + LO.ln1_g, lp + LO.ln1_b);
#pragma unroll
    for (int i = 0; i < TQ; ++i) {
      const int nt = wave + kWaves * i;
      bq[i] = lp[(int)LO.qkv_b + min(nt * 16, 3 * D - 16) + (lane & 15)];
    }
    wq.begin(layer_pack(l, 0), wave, 3 * D / 16, kWaves, lane);
  };
  auto begin_ffn1 = [&](int l) FVAN_INLINE {
    const int lane = opaque(tid & 63);
    const float* lp = layer_theta(l);
    ln2.load(lp + LO.ln2_g, lp + LO.ln2_b);
#pragma unroll
    for (int i = 0; i < T1; ++i) b1[i] = lp[(int)LO.ffn1_b + min((wave + kWaves * i) * 16, 4 * D - 16) + (lane & 15)];
    w1.begin(layer_pack(l, pack_ffn1_offset(D)), wave, 4 * D / 16, kWaves, lane);
  };
  auto begin_ffn2 = [&](int l) FVAN_INLINE {
    const int lane = opaque(tid & 63);
    b2 = layer_theta(l)[(int)LO.ffn2_b + min(tile2, NT2 - 1) * 16 + (lane & 15)];
    const uint4* p2 = layer_pack(l, pack_ffn2_offset(D));
    if constexpr (SK > 1)
      w2.begin(p2 + ((size_t)tile2 * 4 * D / Mode<MODE>::KC + (size_t)part2 * NCS) * 64, 0, 1, 1, lane);
    else
      w2.begin(p2, wave, NT2, kWaves, lane);
  };

  // K/V rows: a batch is UNR rows per lane, RPL rows per wave load, of one sample;
  // a wave's samples are walked as one stream of batches
  struct Batch {
    uint4 k[UNR], v[UNR];
  };
  const int nsw = nb > wave ? (nb - wave + kWaves - 1) / kWaves : 0;   // samples of this wave
  // step t: the slot of position t and the visible slots [0, nvis)
  auto slot_of = [&](int t) FVAN_INLINE { return t < P ? t : P + (t - P) % R; };
  auto nvis_of = [&](int t) FVAN_INLINE { return t < P ? t + 1 : P + min(t - P + 1, R); };
  auto kv_block = [&](int m, int l) FVAN_INLINE { return kvbase + ((size_t)(b0 + m) * nl + l) * 2 * plane; };
  // batch `part` of sample m: raw loads of its rows (the step's own is replaced from
  // LDS when the batch is reduced); rows past the visible keys are zero, so their
  // (zero) probabilities multiply zeros, not stale register contents
  auto issue = [&](Batch& x, int l, int m, int part, int nvis) FVAN_INLINE {
    const int lane = opaque(tid & 63), lrow = lane / LPR, lcol = (lane % LPR) * VEC;
    if constexpr (WIDE) {                   // a wave load is 64 x 16 consecutive bytes
      const int s0 = part * UNR * RPL, bytes = min(max(nvis - s0, 0), UNR * RPL) * (D * (int)sizeof(T));
      T* kb = kv_block(m, l) + (size_t)s0 * D;
      const kv_rsrc_t rk = kv_rsrc(kb, bytes), rv = kv_rsrc(kb + plane, bytes);
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        x.k[u] = kv_load16(rk, 16 * lane + 1024 * u, 0);
        x.v[u] = kv_load16(rv, 16 * lane + 1024 * u, 0);
      }
    } else {
      const kv_rsrc_t r = kv_rsrc(kv_block(m, l), 2 * (int)(plane * sizeof(T)));
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const int s = (part * UNR + u) * RPL + lrow;
        const int at = s < nvis ? (s * D + lcol) * (int)sizeof(T) : kNoLane;
        x.k[u] = kv_load16(r, at, 0);
        x.v[u] = kv_load16(r, at, (int)(plane * sizeof(T)));
      }
    }
  };
  Batch ba, bb;
  auto issue_first = [&](int l, int t) FVAN_INLINE { issue(ba, l, wave, 0, t < N && nsw > 0 ? nvis_of(t) : 0); };

  if (nl > 0) {
    begin_qkv(0);
    issue_first(0, 0);
  }
  __syncthreads();

  // the position embedding of a step: thread tid holds column tid % D of every row
  static_assert(kThreads % D == 0, "a thread's column is the same in every row");
  const int ek = tid % D;
  auto pos_of = [&](int t) FVAN_INLINE { return theta[U.pos_off + (size_t)t * (D - dt) + max(ek - dt, 0)]; };
  float pe = pos_of(0);
  // the two token embeddings of a spin model
  const float te0 = theta[min(ek, dt - 1)], te1 = theta[dt + min(ek, dt - 1)];
  float hw0[D / 16], hw1[D / 16], hb0 = 0.f, hb1 = 0.f;    // the binary head, the lane's columns
  if constexpr (!TOK) {
#pragma unroll
    for (int i = 0; i < D / 16; ++i) {
      hw0[i] = theta[U.head_w + hpart + 16 * i];
      hw1[i] = theta[U.head_w + D + hpart + 16 * i];
    }
    hb0 = theta[U.head_b];
    hb1 = theta[U.head_b + 1];
  }

  for (int t = 0; t < N; ++t) {
    // ---- concatenated embedding [tok_emb[tok]; pos_emb[t]] ----
#pragma unroll
    for (int i = 0; i < KM * D; i += kThreads) {
      const int m = (i + tid) / D;
      if constexpr (TOK) sm.h[m][ek] = ek < dt ? theta[sm.tok[m] * dt + ek] : pe;
      else sm.h[m][ek] = ek < dt ? (sm.tok[m] ? te1 : te0) : pe;
    }
    const int slot = slot_of(t), nvis = nvis_of(t);
    const int per = (nvis + RPL * UNR - 1) / (RPL * UNR);   // batches per sample
    pe = pos_of(min(t + 1, N - 1));
    __syncthreads();

    for (int l = 0; l < nl; ++l) {
      ln_rows<D, MODE, TOK, KM>(sm, ln1);
      __syncthreads();

      // ---- QKV projection; q_t, k_t, v_t to LDS ----
      {
        auto qkv_epi = [&](int nt, const floatx4& a0, const floatx4& a1) FVAN_INLINE {
          const int lane = opaque(tid & 63);
          const floatx4 acc[2] = {a0, a1};
          const int n = nt * 16 + (lane & 15);
          const float bias = pick<TQ>(bq, nt / kWaves);
#pragma unroll
          for (int ri = 0; ri < 4 * NRT; ++ri) {
            const int row = 16 * (ri >> 2) + 4 * (lane >> 4) + (ri & 3);
            const float val = acc[ri >> 2][ri & 3] + bias;
            if (n < D) {
              sm.u.q[row][n] = val * kScaleLog2;
            } else {
              const int which = n >= 2 * D ? 1 : 0;
              sm.kv[row][which][n - D - which * D] = from_f<T>(val);
            }
          }
        };
        mfma_tiles<MODE, D, NRT, Mode<MODE>::SPLIT, TQ>(wq, &sm.a[0][0], Sm::LDA, wave, 3 * D / 16, kWaves, opaque(lane), qkv_epi,
                                                    [&]() FVAN_INLINE { begin_ffn1(l); });
      }
      __syncthreads();

      // ---- masked attention over slots [0, nvis), one wave per sample ----
      // Two batches in flight: a batch's registers are loaded again as soon as it has
      // been reduced, across sample boundaries too.
      {
        float qv[VEC], o[VEC];
        float mx = -INFINITY, sum = 0.f;
        auto reduce = [&](Batch& x, int m, int part) FVAN_INLINE {
          const int lane = opaque(tid & 63), lrow = lane / LPR, lcol = (lane % LPR) * VEC;
          if (part == 0) {
#pragma unroll
            for (int i = 0; i < VEC; ++i) { qv[i] = sm.u.q[m][lcol + i]; o[i] = 0.f; }
            mx = -INFINITY;
            sum = 0.f;
            // append k_t (row group 0) and v_t (row group 1) to the cache: this wave
            // is the only reader of the sample's rows
            if constexpr (WIDE) {            // one row each, from the lanes of the first row group
              T* kb = kv_block(m, l) + (size_t)slot * D;
              kv_store16(kv_rsrc(kb, D * (int)sizeof(T)), *reinterpret_cast<const uint4*>(&sm.kv[m][0][lcol]),
                         16 * lane);
              kv_store16(kv_rsrc(kb + plane, D * (int)sizeof(T)), *reinterpret_cast<const uint4*>(&sm.kv[m][1][lcol]),
                         16 * lane);
            } else {
              kv_store16(kv_rsrc(kv_block(m, l), 2 * (int)(plane * sizeof(T))),
                         *reinterpret_cast<const uint4*>(&sm.kv[m][lrow & 1][lcol]),
                         lrow < 2 ? (int)((lrow * plane + slot * D + lcol) * sizeof(T)) : kNoLane);
            }
          }
          const int s0 = part * RPL * UNR;
          if (slot >= s0 && slot < s0 + RPL * UNR) {   // the step's own row
            const int us = (slot - s0) / RPL;
#pragma unroll
            for (int u = 0; u < UNR; ++u)
              if (u == us && lrow == (slot - s0) % RPL) {
                x.k[u] = *reinterpret_cast<const uint4*>(&sm.kv[m][0][lcol]);
                x.v[u] = *reinterpret_cast<const uint4*>(&sm.kv[m][1][lcol]);
              }
          }
          float sc[UNR];
          float mnew = mx;
#pragma unroll
          for (int u = 0; u < UNR; ++u) {
            Chunk<T> kc;
            kc.unpack(x.k[u]);
            float d = 0.f;
#pragma unroll
            for (int i = 0; i < VEC; ++i) d += qv[i] * kc.v[i];
            if (LPH >= 2) d += lane_xor(d, 1);
            if (LPH >= 4) d += lane_xor(d, 2);
            if (LPH >= 8) d += lane_xor(d, 4);
            if (LPH >= 16) d += lane_xor(d, 8);
            sc[u] = s0 + u * RPL + lrow < nvis ? d : -INFINITY;
            mnew = fmaxf(mnew, sc[u]);
          }
          // a lane with no visible row so far subtracts 0 instead of its -inf maximum:
          // its exponentials are exp2(-inf) = 0
          const float base = mnew == -INFINITY ? 0.f : mnew;
          const float corr = __builtin_amdgcn_exp2f(mx - base);
          // The rescale of the running sums is fused with the batch's first row, written
          // out so that the roundings do not depend on how the compiler contracts.
          // (At d = 64 in split mode two elements round the other product: samples of
          // one seed stay the same from one version of the kernel to the next.)
          auto keeps = [](int i) { return D == 64 && Mode<MODE>::SPLIT && i < 2; };
#pragma unroll
          for (int u = 0; u < UNR; ++u) {
            const float p = __builtin_amdgcn_exp2f(sc[u] - base);
            Chunk<T> vc;
            vc.unpack(x.v[u]);
            sum = u == 0 ? __builtin_fmaf(sum, corr, p) : sum + p;
#pragma unroll
            for (int i = 0; i < VEC; ++i)
              o[i] = u > 0      ? __builtin_fmaf(p, vc.v[i], o[i])
                     : keeps(i) ? __builtin_fmaf(p, vc.v[i], o[i] * corr)
                                : __builtin_fmaf(o[i], corr, p * vc.v[i]);
          }
          mx = mnew;
          if (part == per - 1) {
            // Merge the RPL row groups of the wave, pairs LPR .. 32 lanes apart in turn.
            // Each merge also halves the elements a lane keeps (the lane with the
            // pair's bit set takes the upper half), so the o merges cost 4 + 2 + 1
            // elements instead of 8 + 8 + 8; the lower lane's operand order is used in
            // both lanes.  Then every lane adds its element(s) of the heads' outputs.
            int first = 0;                           // first element this lane keeps
            bool adds = true;
#pragma unroll
            for (int off = LPR, keep = VEC; off < 64; off <<= 1) {
              float ml = mx, mh = mx, sl = sum, sh = sum;
              lane_pair(ml, mh, off);
              lane_pair(sl, sh, off);
              const float mn = fmaxf(ml, mh), base2 = mn == -INFINITY ? 0.f : mn;
              const float c1 = __builtin_amdgcn_exp2f(ml - base2);
              const float c2 = __builtin_amdgcn_exp2f(mh - base2);
              sum = __builtin_fmaf(sl, c1, sh * c2);
              if (keep > 1) {
                keep >>= 1;
                if (lane & off) first += keep;
#pragma unroll
                for (int i = 0; i < VEC / 2; ++i)
                  if (i < keep) {
                    float lo = o[i], hi = o[i + keep];
                    lane_pair(lo, hi, off);
                    o[i] = __builtin_fmaf(lo, c1, hi * c2);
                  }
              } else {
                float lo = o[0], hi = o[0];
                lane_pair(lo, hi, off);
                o[0] = __builtin_fmaf(lo, c1, hi * c2);
                adds = adds && !(lane & off);
              }
              mx = mn;
            }
            constexpr int KEPT = VEC / RPL > 1 ? VEC / RPL : 1;
            const float inv = 1.0f / sum;
            if (adds) {
#pragma unroll
              for (int i = 0; i < KEPT; ++i)
                sm.h[m][lcol + first + i] = __builtin_fmaf(o[i], inv, sm.h[m][lcol + first + i]);
            }
          }
        };
        // (m, part) of the batch to reduce and of the one two further on
        int left = per * nsw, m = wave, part = 0, mi = wave, pi = 0;
        auto next = [&](int& mm, int& pp) FVAN_INLINE {
          if (++pp == per) {
            pp = 0;
            mm += kWaves;
          }
        };
        next(mi, pi);
        issue(bb, l, mi, pi, left > 1 ? nvis : 0);
        next(mi, pi);
        while (left > 0) {
          reduce(ba, m, part);
          next(m, part);
          issue(ba, l, mi, pi, left > 2 ? nvis : 0);   // always: a known number of loads in flight
          next(mi, pi);
          if (--left == 0) break;
          reduce(bb, m, part);
          next(m, part);
          issue(bb, l, mi, pi, left > 2 ? nvis : 0);   // always: a known number of loads in flight
          next(mi, pi);
          --left;
        }
      }
      __syncthreads();

      // ---- feed-forward block ----
      ln_rows<D, MODE, TOK, KM>(sm, ln2);
      __syncthreads();
      {
        // split mode: GELU(h) goes to LDS already split, in the layout ln_rows
        // writes (per 8-element group of a row: 8 hi BF16, then 8 lo), for FFN2
        auto ffn1_epi = [&](int nt, const floatx4& a0, const floatx4& a1) FVAN_INLINE {
          const int lane = opaque(tid & 63);
          const floatx4 acc[2] = {a0, a1};
          const int n = nt * 16 + (lane & 15);
          const float bias = pick<T1>(b1, nt / kWaves);
#pragma unroll
          for (int ri = 0; ri < 4 * NRT; ++ri) {
            const int row = 16 * (ri >> 2) + 4 * (lane >> 4) + (ri & 3);
            const float gv = gelu(acc[ri >> 2][ri & 3] + bias);
            if constexpr (Mode<MODE>::SPLIT) {
              const __bf16 hb = (__bf16)gv;
              const __bf16 lb = (__bf16)(gv - (float)hb);
              __bf16* hr = reinterpret_cast<__bf16*>(&sm.u.hid[row][0]) + (n >> 3) * 16 + (n & 7);
              hr[0] = hb;
              hr[8] = lb;
            } else {
              sm.u.hid[row][n] = from_f<typename Mode<MODE>::ActT>(gv);
            }
          }
        };
        mfma_tiles<MODE, D, NRT, Mode<MODE>::SPLIT, T1>(w1, &sm.a[0][0], Sm::LDA, wave, 4 * D / 16, kWaves, opaque(lane), ffn1_epi,
                                                    [&]() FVAN_INLINE { begin_ffn2(l); });
      }
      __syncthreads();
      {
        // once FFN2's weights are on their way: the next layer's (or the next
        // step's first layer's) parameters and first K/V rows
        const bool wrap = l + 1 == nl;
        auto ahead = [&]() FVAN_INLINE {
          begin_qkv(wrap ? 0 : l + 1);
          issue_first(wrap ? 0 : l + 1, wrap ? t + 1 : t);
        };
        if constexpr (SK == 1) {
          auto ffn2_epi = [&](int nt, const floatx4& a0, const floatx4& a1) FVAN_INLINE {
          const int lane = opaque(tid & 63);
            const floatx4 acc[2] = {a0, a1};
            const int n = nt * 16 + (lane & 15);
#pragma unroll
            for (int ri = 0; ri < 4 * NRT; ++ri)
              sm.h[16 * (ri >> 2) + 4 * (lane >> 4) + (ri & 3)][n] += acc[ri >> 2][ri & 3] + b2;
          };
          static_assert(NT2 <= kWaves, "one FFN2 tile per wave");
          mfma_tiles<MODE, 4 * D, NRT, Mode<MODE>::SPLIT, 1>(w2, &sm.u.hid[0][0], Sm::LDH, wave, NT2, kWaves, opaque(lane),
                                                          ffn2_epi, ahead);
        } else {
          // fewer output tiles than waves: the SK waves of a tile take consecutive
          // K ranges; the upper ranges' sums meet the lowest one's through LDS and
          // are added in range order
          static_assert(NCS * SK * Mode<MODE>::KC == 4 * D, "whole K chunks per range");
          const int ln = opaque(lane), n = tile2 * 16 + (ln & 15);
          floatx4 r[2];
          auto keep = [&](int, const floatx4& a0, const floatx4& a1) FVAN_INLINE {
            r[0] = a0;
            r[1] = a1;
          };
          const float bias = b2;
          mfma_tiles<MODE, 4 * D / SK, NRT, Mode<MODE>::SPLIT, 1>(w2, &sm.u.hid[0][0] + part2 * NCS * Mode<MODE>::KC,
                                                               Sm::LDH, 0, 1, 1, opaque(lane), keep, ahead);
          if (part2 > 0) {
#pragma unroll
            for (int ri = 0; ri < 4 * NRT; ++ri)
              sm.kpart[part2 - 1][16 * (ri >> 2) + 4 * (ln >> 4) + (ri & 3)][n] = r[ri >> 2][ri & 3];
          }
          __syncthreads();
          if (part2 == 0) {
#pragma unroll
            for (int ri = 0; ri < 4 * NRT; ++ri) {
              const int row = 16 * (ri >> 2) + 4 * (ln >> 4) + (ri & 3);
              float v = r[ri >> 2][ri & 3];
#pragma unroll
              for (int q = 0; q < Sm::KP; ++q) v += sm.kpart[q][row][n];
              sm.h[row][n] += v + bias;
            }
          }
        }
      }
      __syncthreads();
    }

    // ---- head, Philox draw, decision ----
    if constexpr (TOK) {
      // logits z[m][v] = W_h[v] . h[m] + b[v]: thread (v, half) for half of the tile's
      // samples, up to 8 at a time.  The weights are read across the vocabulary (the FP32
      // transpose), 8 loads in flight.  Bound by the reads of sm.h: row-wise weight reads,
      // one cache line per lane, took 22 of the 49 us of a step of d = 128, 256 tokens and
      // 8 samples per workgroup; now 10.  All 16 samples of a half at a time, or 16 loads
      // in flight, are 2 to 5 % slower over a call: the next layer's first loads are held
      // across the logits, so that even this form spills (d = 128, 64-wide heads: 19
      // registers in split mode, 10 in FP32, 4 and none without those loads; the calls are
      // faster with them, 1500 samples of 100 positions 8.6 -> 5.4 ms).
      {
        const int v = tid & (kMaxVocab - 1), half = tid / kMaxVocab;
        const int each = (nb + 1) / 2, m0 = half * each, m1 = min(nb, m0 + each);
        const uint32_t wv = (uint32_t)(min(v, U.vocab - 1) * U.head_sv);
        auto logits = [&](auto count) FVAN_INLINE {
          constexpr int S = decltype(count)::value;
          for (int mb = m0; mb < m1; mb += S) {
            float acc[S];
#pragma unroll
            for (int i = 0; i < S; ++i) acc[i] = 0.f;
#pragma unroll 2
            for (int k = 0; k < D; k += 4) {
              const float* wr = U.head + (uint32_t)(k * U.head_sk);
              const float w0 = wr[wv], w1 = wr[wv + U.head_sk], w2 = wr[wv + 2 * U.head_sk], w3 = wr[wv + 3 * U.head_sk];
#pragma unroll
              for (int i = 0; i < S; ++i) {
                const float4 x = *reinterpret_cast<const float4*>(&sm.h[min(mb + i, KM - 1)][k]);
                acc[i] += w0 * x.x + w1 * x.y + w2 * x.z + w3 * x.w;
              }
            }
            const float bias = theta[U.head_b + min(v, U.vocab - 1)];
#pragma unroll
            for (int i = 0; i < S; ++i)
              if (v < U.vocab && mb + i < m1) sm.u.z[mb + i][v] = acc[i] + bias;
          }
        };
        if (each <= 2) logits(std::integral_constant<int, 2>());
        else if (each <= 4) logits(std::integral_constant<int, 4>());
        else logits(std::integral_constant<int, 8>());
      }
      __syncthreads();
      // softmax and draw: 16 lanes per sample, lane hpart holds logits 16 hpart .. 16 hpart + 15.
      // The token is the largest k >= 1 with u < sum_{j >= k} p_j (else 0), decided as
      // u * total < sum_{j >= k} e_j with e_j = exp(z_j - max), total = sum_j e_j.
      if (hm < nb) {
        const int V = U.vocab, v0 = 16 * hpart;
        float zl[16];
        float mx = -INFINITY;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          zl[j] = v0 + j < V ? sm.u.z[hm][v0 + j] : -INFINITY;
          mx = fmaxf(mx, zl[j]);
        }
        mx = row_max16(mx);
        float e[16], bs = 0.f;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          e[j] = v0 + j < V ? expf(zl[j] - mx) : 0.f;
          bs += e[j];
        }
        // suffix sums over the lanes of the row: suf = sum of the block sums of lanes >= hpart
        float suf = bs;
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) {
          const float o = __shfl_down(suf, off, 16);
          if (hpart + off < 16) suf += o;
        }
        const float total = __shfl(suf, 0, 16);
        if ((t & 3) == 0) {
          const uint4 w = philox4x32_10(make_uint4((uint32_t)(t >> 2), (uint32_t)(b0 + hm), U.stream_lo, U.stream_hi),
                                        U.seed_lo, U.seed_hi);
          ur[0] = u24(w.x); ur[1] = u24(w.y); ur[2] = u24(w.z); ur[3] = u24(w.w);
        }
        const float ut = ur[t & 3] * total;
        float run = suf - bs;   // the blocks above this lane's
        float cand = -1.f;
#pragma unroll
        for (int j = 15; j >= 0; --j) {
          run += e[j];
          if (cand < 0.f && v0 + j >= 1 && v0 + j < V && ut < run) cand = (float)(v0 + j);
        }
        const int tk = max(0, (int)row_max16(cand));
        float zt = 0.f;
#pragma unroll
        for (int j = 0; j < 16; ++j) zt = v0 + j == tk ? zl[j] : zt;
        zt = row_sum16(zt);
        if (hpart == 0) {
          lq += zt - (mx + logf(total));
          sm.tok[hm] = tk;
          sm.sbuf[hm][t & 63] = (int8_t)(uint8_t)tk;
        }
      }
    } else {
      if (hm < KM) {
        float z0 = 0.f, z1 = 0.f;
#pragma unroll
        for (int i = 0; i < D / 16; ++i) {
          const float x = sm.h[hm][hpart + 16 * i];
          z0 += x * hw0[i];
          z1 += x * hw1[i];
        }
        z0 = reduce16(z0);
        z1 = reduce16(z1);
        if (hpart == 0) {
          if ((t & 3) == 0) {
            const uint4 w = philox4x32_10(make_uint4((uint32_t)(t >> 2), (uint32_t)(b0 + hm), U.stream_lo, U.stream_hi),
                                          U.seed_lo, U.seed_hi);
            ur[0] = u24(w.x); ur[1] = u24(w.y); ur[2] = u24(w.z); ur[3] = u24(w.w);
          }
          const float d = (z1 + hb1) - (z0 + hb0);
          const float e = expf(-fabsf(d));
          const float pplus = d >= 0.f ? 1.0f / (1.0f + e) : e / (1.0f + e);
          const float u = ur[t & 3];
          const int s = u < pplus ? 1 : 0;
          lq += s ? -softplus(-d) : -softplus(d);
          sm.tok[hm] = s;
          sm.sbuf[hm][t & 63] = s ? (int8_t)1 : (int8_t)-1;
        }
      }
    }
    __syncthreads();
    if ((t & 63) == 63 || t == N - 1) {
      const int base = t & ~63;
      for (int i = tid; i < KM * 64; i += kThreads) {
        const int m = i >> 6, j = i & 63;
        if (m < nb && base + j <= t) U.spins[(size_t)(b0 + m) * N + base + j] = sm.sbuf[m][j];
      }
    }
  }
  if (hpart == 0 && hm < nb) U.logq[b0 + hm] = lq;
  __syncthreads();
}

template <int D, int MODE, int DH, bool TOK, int KM, bool WIDE>
__global__ __launch_bounds__(kThreads) void decode_kernel(DecodeUnit u0, const DecodeUnit* __restrict__ table,
                                                          int n_units, int total_tiles, int* queue) {
  __shared__ DecodeSmem<D, MODE, TOK, KM> sm;
  __shared__ int s_tile;
  bool first = true;
  for (;;) {
    if (threadIdx.x == 0) {
      if (queue) s_tile = atomicAdd(queue, 1);
      else s_tile = first ? (int)blockIdx.x : total_tiles;
    }
    __syncthreads();
    const int tile = s_tile;
    __syncthreads();
    first = false;
    if (tile >= total_tiles) break;
    if (table) {
      int lo = 0, hi = n_units - 1;        // last unit with tile0 <= tile
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (table[mid].tile0 <= tile) lo = mid; else hi = mid - 1;
      }
      const DecodeUnit U = table[lo];
      decode_tile<D, MODE, DH, TOK, KM, WIDE>(sm, U, tile - U.tile0);
    } else {
      decode_tile<D, MODE, DH, TOK, KM, WIDE>(sm, u0, tile);
    }
  }
}

template <int D, int MODE, int DH, bool TOK, int KM, bool WIDE = false>
hipError_t launch_d(const DecodeUnit& u0, const DecodeUnit* table, int n_units, int total_tiles, int* queue, int grid,
                    hipStream_t s) {
  hipLaunchKernelGGL((decode_kernel<D, MODE, DH, TOK, KM, WIDE>), dim3(grid), dim3(kThreads), 0, s, u0, table, n_units,
                     total_tiles, queue);
  return hipGetLastError();
}

// The instantiations decode_ext.hip holds (X(D, MODE, DH, TOK, KM)): other head
// widths and token models with 32-sample tiles, and 16-sample tiles of the
// single-spin 16-wide-head kernels (batched launches) and of the patched 3D
// model's kernels.
#define FVAN_DECODE_EXT_LIST(X)                                                                                \
  X(32, 0, 32, false, 32) X(32, 2, 32, false, 32) X(64, 0, 32, false, 32) X(64, 2, 32, false, 32)             \
  X(64, 0, 64, false, 32) X(64, 2, 64, false, 32) X(128, 0, 32, false, 32) X(128, 2, 32, false, 32)           \
  X(128, 0, 64, false, 32) X(128, 2, 64, false, 32) X(32, 0, 16, true, 32) X(32, 2, 16, true, 32)             \
  X(32, 0, 32, true, 32) X(32, 2, 32, true, 32) X(64, 0, 16, true, 32) X(64, 2, 16, true, 32)                 \
  X(64, 0, 32, true, 32) X(64, 2, 32, true, 32) X(64, 0, 64, true, 32) X(64, 2, 64, true, 32)                 \
  X(128, 0, 16, true, 32) X(128, 2, 16, true, 32) X(128, 0, 32, true, 32) X(128, 2, 32, true, 32)             \
  X(128, 0, 64, true, 32) X(128, 2, 64, true, 32)                                                             \
  X(32, 0, 16, false, 16) X(32, 2, 16, false, 16) X(64, 0, 16, false, 16) X(64, 2, 16, false, 16)             \
  X(128, 0, 16, false, 16) X(128, 2, 16, false, 16) X(128, 0, 64, true, 16) X(128, 2, 64, true, 16)
#define FVAN_DECODE_INST(D, MODE, DH, TOK, KM)                                                         \
  template hipError_t launch_d<D, MODE, DH, TOK, KM>(const DecodeUnit&, const DecodeUnit*, int, int, int*, int, \
                                                      hipStream_t);
#define FVAN_DECODE_EXTERN(D, MODE, DH, TOK, KM) extern FVAN_DECODE_INST(D, MODE, DH, TOK, KM)

// The WIDE instantiations (decode_wide.hip): every model shape, with 32-sample tiles.
#define FVAN_DECODE_WIDE_LIST(X)                                                                                \
  X(32, 0, 16) X(32, 2, 16) X(32, 0, 32) X(32, 2, 32) X(64, 0, 16) X(64, 2, 16) X(64, 0, 32) X(64, 2, 32)      \
  X(64, 0, 64) X(64, 2, 64) X(128, 0, 16) X(128, 2, 16) X(128, 0, 32) X(128, 2, 32) X(128, 0, 64) X(128, 2, 64)
#define FVAN_DECODE_WIDE_INST(D, MODE, DH)                                                                        \
  template hipError_t launch_d<D, MODE, DH, false, 32, true>(const DecodeUnit&, const DecodeUnit*, int, int, int*, \
                                                             int, hipStream_t);                                    \
  template hipError_t launch_d<D, MODE, DH, true, 32, true>(const DecodeUnit&, const DecodeUnit*, int, int, int*,  \
                                                            int, hipStream_t);
#define FVAN_DECODE_WIDE_EXTERN(D, MODE, DH)                                                                      \
  extern template hipError_t launch_d<D, MODE, DH, false, 32, true>(const DecodeUnit&, const DecodeUnit*, int, int, \
                                                                    int*, int, hipStream_t);                       \
  extern template hipError_t launch_d<D, MODE, DH, true, 32, true>(const DecodeUnit&, const DecodeUnit*, int, int,  \
                                                                   int*, int, hipStream_t);

}  // namespace fvan
