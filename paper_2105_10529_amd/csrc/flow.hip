// Coupling normalising flow (piecewise-quadratic coupling layers, Mueller et
// al. 2019) on gfx950: forward/inverse layer kernel, backward kernels, Adam,
// and the flow part of the C ABI.
//
// Kernels:
//   k_coupling      all coupling layers for a tile of 64 events; of each the
//                   three dense layers as BF16 MFMA products (v_mfma_f32_16x16x32_bf16,
//                   FP32 accumulation) with the hidden activations resident in
//                   LDS, then the FP32 piecewise-quadratic CDF (or its inverse)
//                   of each transformed coordinate; optionally keeps the layer
//                   input for the backward pass
//   k_backward      the backward pass through all layers for a tile of 64
//                   events; of each the forward products again, the derivatives
//                   of the PQ transforms, and the activation-gradient products;
//                   writes the operands of the weight gradients
//   k_wgrad         the weight-gradient products of all layers, split over events
//   k_reduce_grad   ordered reduction of their partials into the FP32 gradient
//   k_adam          Adam on the FP32 masters and refresh of the BF16 copies
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <vector>

#include "../../include/mf_flow.h"
#include "flow_internal.h"
#include "pipeline.h"
#include "status.h"

namespace mf {
namespace flow {

constexpr int H = 256;        // hidden width
constexpr int KB = 32;        // PQ bins
constexpr int NO = 2 * KB + 1;  // logits per transformed coordinate
constexpr int NOP = 80;       // NO padded: stride of a coordinate's output biases and of its k range in W3q
constexpr int NOG = 72;       // NO padded to 16-byte chunks: logit gradients of one coordinate
constexpr int KA = 32;        // first-layer k width: inputs split as BF16 hi (k < 16) + lo (k >= 16)
constexpr int KLO = 16;       // offset of the low parts
constexpr int T = 64;         // events per workgroup of the layer kernel
constexpr int LDO = 68;       // LDS row stride (floats) of one coordinate's 64 leading logits (16-byte rows)
constexpr int FMAXD = 16;
constexpr int TBMAX = FMAXD / 2;  // transformed coordinates per layer (the masks take one half)
constexpr int MAXL = 8;
constexpr float SLOPE = 0.01f;

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct LayerDev {
  int dA, dB;
  int a_idx[FMAXD];
  int b_idx[FMAXD];
  const bf16* W1t;   // [H][KA]      (W1 transposed, at k = i and k = KLO + i)
  const float* b1;   // [H]
  const float* b2;   // [H]
  const float* b3p;  // [dB*NOP]
  // The coupling kernel's A fragments of the second layer and of the 64
  // leading logits of the third, packed so that one wave's fragment load is
  // 1 KB of consecutive bytes (64 lanes x 16 B) instead of 16 rows x 64 B;
  // element (k, j) is W[k][j] (input k, output j; the outputs of W3 padded
  // to NOP per coordinate):
  //   W2p[((w * 8 + ks) * 4 + jt) * 64 + lane][8]:  output j = 64 w + 16 jt + (lane & 15),
  //                                                 k = 32 ks + 8 (lane >> 4) + e
  //   W3p[((c * 4 + w) * 8 + ks) * 64 + lane][8]:  output c NOP + 16 w + (lane & 15), same k
  //   W3L[ks * 64 + lane][8]:                    output (lane & 15) NOP + 2K (the 65th
  //                                                 logit of coordinate lane & 15; zero
  //                                                 past d_B), same k
  const bf16* W2p;   // [H][H]
  const bf16* W3p;   // [dB][64][H]
  const bf16* W3L;   // [16][H]
  // The backward products' A fragments, packed in the same way with the roles
  // of inputs and outputs exchanged:
  //   W2q[((w * 8 + ks) * 4 + jt) * 64 + lane][8]:  W2[j][k], j = 64 w + 16 jt + (lane & 15),
  //                                                 k = 32 ks + 8 (lane >> 4) + e
  //   W3q[((ks * 4 + w) * 4 + jt) * 64 + lane][8]: column k of W3 with NOP columns per coordinate,
  //                                                 c NOP + r (zero for r >= NO), same j and k
  //   W1q[ks * 64 + lane][8]:                       W1[lane & 15][k] (zero rows past d_A)
  const bf16* W2q;   // [H][H]
  const bf16* W3q;   // [dB NOP rounded up to 32][H]
  const bf16* W1q;   // [16][H]
};

struct Layers {
  LayerDev L[MAXL];
};

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Hidden activations in LDS: [T][H] bf16 with the 16-byte chunks of a row
// permuted by the row index, so that the 16 rows read by one fragment load
// fall in different banks.
__device__ __forceinline__ int hs(int m, int k) { return m * H + ((((k >> 3) ^ (m & 15))) << 3) + (k & 7); }

// The median of (v, 0.01 v, FLT_MAX) is max(v, 0.01 v) for finite v: v for v >= 0 and 0.01 v
// below, the LeakyReLU in two operations (fmaxf would add a canonicalising
// instruction per input in IEEE mode)
__device__ __forceinline__ float leaky(float v) { return __builtin_amdgcn_fmed3f(v, SLOPE * v, 3.40282347e38f); }

// Exchanges inside an aligned group of four lanes through DPP quad
// permutations (no LDS round trip): lane ^ 1, lane ^ 2, and the group's lane
// 0, 1 or 2 broadcast to all four.  A quad permutation reads a lane of the
// same group for every lane, so no old value is needed.
constexpr int QX1 = 0xB1, QX2 = 0x4E, QB0 = 0x00, QB1 = 0x55, QB2 = 0xAA;
template <int CTRL> __device__ __forceinline__ float qdpp(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, true));
}
template <int CTRL> __device__ __forceinline__ int qdpp(int x) {
  return __builtin_amdgcn_mov_dpp(x, CTRL, 0xF, 0xF, true);
}
// max(a, b) of finite values as the median of (a, b, FLT_MAX), without the
// canonicalising instructions fmaxf adds in IEEE mode
__device__ __forceinline__ float max_nc(float a, float b) {
  return __builtin_amdgcn_fmed3f(a, b, 3.40282347e38f);
}

// ------------------------------------------------------------ PQ transform
// Epilogue of a transposed dense layer: acc[jt][mt][i] is feature
// 64 wave + 16 jt + 4 quad + i of event 16 mt + row, bias included (it is
// the accumulator's initial value); applies the LeakyReLU, rounds to BF16 and
// stores the four features with one 8-byte write into the permuted [T][H]
// activation tile.
__device__ __forceinline__ void store_features(bf16* h, const f32x4 (&acc)[4][4], int wave, int row, int quad) {
#pragma unroll
  for (int jt = 0; jt < 4; ++jt) {
    const int f0 = 64 * wave + 16 * jt + 4 * quad;
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      bf16x4 v;
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = (bf16)leaky(acc[jt][mt][i]);
      *reinterpret_cast<bf16x4*>(h + hs(16 * mt + row, f0)) = v;
    }
  }
}

// The bias of the four features 64 wave + 16 jt + 4 quad + i (i = 0..3) as an
// accumulator tile.
__device__ __forceinline__ f32x4 bias4(const float* __restrict__ b, int wave, int jt, int quad) {
  const float* p = b + 64 * wave + 16 * jt + 4 * quad;
  return f32x4{p[0], p[1], p[2], p[3]};
}

// The PQ transform of one coordinate with four lanes per event: lane part p
// holds the bins [8p, 8p+8) and the vertices [8p, 8p+8] of the 2K+1 logits
// (the first 2K in LDS at o, the last one, vlast, in a register of the
// p = 3 lane); maxima, sums, prefix offsets and the bin's owner are combined
// with DPP quad exchanges.  Same bin rule as find_bin: the largest k >= 1
// whose left edge (running width, or running area for the sampling
// direction) is <= t, else 0.  Every lane of the group returns the result
// (y or z) and the density.  Reciprocals use the hardware approximation
// (1 ulp).
template <bool INVERSE>
__device__ __forceinline__ void pq_quad(const float* o, float vlast, float t, int p, float& res, float& pdf) {
  constexpr int KP = KB / 4;
  float w[KP], v[KP + 1];
#pragma unroll
  for (int k = 0; k < KP; ++k) w[k] = o[KP * p + k];
#pragma unroll
  for (int k = 0; k < KP; ++k) v[k] = o[KB + KP * p + k];
  {
    // the part's last vertex: the next part's first, or the 2K+1-th logit
    const float vn = o[KB + KP * p + (p < 3 ? KP : 0)];
    v[KP] = p < 3 ? vn : vlast;
  }
  // exp(x - m) as 2^(x log2 e - m log2 e), one FMA and the hardware exp2
  constexpr float L2E = 1.4426950408889634f;
  float mw = w[0];
#pragma unroll
  for (int k = 1; k < KP; ++k) mw = fmaxf(mw, w[k]);
  mw = max_nc(mw, qdpp<QX1>(mw));
  mw = max_nc(mw, qdpp<QX2>(mw));
  const float mwl = mw * L2E;
  // the widths stay unnormalised (sum sw); the part's sum is its offset
  float sw = 0.0f;
#pragma unroll
  for (int k = 0; k < KP; ++k) {
    w[k] = __builtin_amdgcn_exp2f(fmaf(w[k], L2E, -mwl));
    sw += w[k];
  }
  const float part_w = sw;
  sw += qdpp<QX1>(sw);
  sw += qdpp<QX2>(sw);
  float mv = v[0];
#pragma unroll
  for (int k = 1; k <= KP; ++k) mv = fmaxf(mv, v[k]);
  mv = max_nc(mv, qdpp<QX1>(mv));
  mv = max_nc(mv, qdpp<QX2>(mv));
  const float mvl = mv * L2E;
#pragma unroll
  for (int k = 0; k <= KP; ++k) v[k] = __builtin_amdgcn_exp2f(fmaf(v[k], L2E, -mvl));
  // bin areas with the unnormalised widths and heights, twice over:
  // ar_k = (v_k + v_k+1) w_k, total nl
  float ar[KP];
  float nl = 0.0f;
#pragma unroll
  for (int k = 0; k < KP; ++k) {
    ar[k] = (v[k] + v[k + 1]) * w[k];
    nl += ar[k];
  }
  const float part_a = nl;
  nl += qdpp<QX1>(nl);
  nl += qdpp<QX2>(nl);
  // normalised: width w_k / sw, area ar_k / nl, height v_k 2 sw / nl (unit
  // total area); the running edges are compared in unnormalised units
  const float isw = __builtin_amdgcn_rcpf(sw);
  const float iar = __builtin_amdgcn_rcpf(nl);
  const float tt = t * (INVERSE ? nl : sw);
  // exclusive offsets of the running width and area at the part's first bin
  const float s0 = qdpp<QB0>(part_w), s1 = qdpp<QB1>(part_w), s2 = qdpp<QB2>(part_w);
  const float a0 = qdpp<QB0>(part_a), a1 = qdpp<QB1>(part_a), a2 = qdpp<QB2>(part_a);
  float S = (p > 0 ? s0 : 0.0f) + (p > 1 ? s1 : 0.0f) + (p > 2 ? s2 : 0.0f);
  float A = (p > 0 ? a0 : 0.0f) + (p > 1 ? a1 : 0.0f) + (p > 2 ? a2 : 0.0f);
  // the edges grow with the bin index, so bin b is owned by the last lane
  // of the group whose first bin is taken
  const bool first = p == 0 || (INVERSE ? A : S) <= tt;
  int owner = first ? p : -1;
  float Sb = S, Ab = A, Wb = w[0], Vb = v[0], Vb1 = v[1];
  S += w[0];
  A += ar[0];
#pragma unroll
  for (int k = 1; k < KP; ++k) {
    const bool take = (INVERSE ? A : S) <= tt;
    Sb = take ? S : Sb;
    Ab = take ? A : Ab;
    Wb = take ? w[k] : Wb;
    Vb = take ? v[k] : Vb;
    Vb1 = take ? v[k + 1] : Vb1;
    S += w[k];
    A += ar[k];
  }
  owner = max(owner, qdpp<QX1>(owner));
  owner = max(owner, qdpp<QX2>(owner));
  Sb *= isw;
  Ab *= iar;
  Wb *= isw;
  const float hn = 2.0f * sw * iar;
  Vb *= hn;
  Vb1 *= hn;
  const float dV = Vb1 - Vb;
  const float iW = __builtin_amdgcn_rcpf(Wb);
  float r, q;
  if (!INVERSE) {
    const float al = fminf(fmaxf((t - Sb) * iW, 0.0f), 1.0f);
    r = Ab + Wb * (al * Vb + 0.5f * al * al * dV);
    q = Vb + al * dV;
  } else {
    const float cc = (t - Ab) * iW;
    const float disc = fmaxf(Vb * Vb + 2.0f * dV * cc, 0.0f);
    // hardware square root (1 ulp)
    float al = 2.0f * cc * __builtin_amdgcn_rcpf(Vb + __builtin_amdgcn_sqrtf(disc));
    al = fminf(fmaxf(al, 0.0f), 1.0f);
    r = Sb + al * Wb;
    q = Vb + al * dV;
  }
  // only the owner of bin b holds the right values: a sum over the group
  // with the other three lanes contributing exact zeros
  const bool own = owner == p;
  float rr = own ? r : 0.0f, qq = own ? q : 0.0f;
  rr += qdpp<QX1>(rr);
  qq += qdpp<QX1>(qq);
  res = rr + qdpp<QX2>(rr);
  pdf = qq + qdpp<QX2>(qq);
}

// A copy of x whose value the compiler does not follow: LDS offsets derived
// from it are computed where they are used instead of being kept in registers
// from one phase of a kernel to the next (9 spilled registers otherwise in
// k_coupling, 123 in k_backward).
__device__ __forceinline__ int fresh(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// -------------------------------------------------------- coupling layers
// All nl layers for events [64 blockIdx.x, +64): y is [d][ld] (n <= ld events
// used) and is transformed in place (a layer's kept coordinates are only
// read).  INVERSE selects the sampling direction, in which the last layer
// comes first.  logq[e] is set to the sum over the layers.  CACHE keeps the
// input points of layer l in lin + l lstride, [d][n].
//
// A tile needs no other tile between its layers, so one launch runs them all:
// a layer of few events is a chain of latencies, and of many events has a last
// round of tiles that is not full.  6 layers, one launch per layer and one for
// all: 700 points of 7 dimensions 68 and 60 us of kernels, 1e6 points of 10
// dimensions 2.25 and 2.21 ms.
//
// LDS: one [T][H] BF16 tile that holds the first hidden layer and then the
// second (written over the first once every wave has read it), and one
// [T][LDO] FP32 tile for the 64 leading logits of the current coordinate
// (before that, its first 4 KB hold the first-layer inputs), and the inputs
// of the transformed coordinates (2 KiB): 51.0 KiB, so that three
// workgroups share a compute unit.
template <bool INVERSE, bool CACHE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) k_coupling(Layers layers, int nl, float* __restrict__ y, int64_t n, int64_t ld,
                                                  float* __restrict__ logq, float* __restrict__ lin, int64_t lstride, int d) {
  __shared__ __attribute__((aligned(16))) bf16 h[T * H];
  __shared__ __attribute__((aligned(16))) float out[T * LDO];
  __shared__ float tb[TBMAX * T];
  static_assert(T * KA * sizeof(bf16) <= T * LDO * sizeof(float), "first-layer inputs must fit the logit tile");
  bf16* xa = reinterpret_cast<bf16*>(out);  // [T][KA]
  // the wave index is uniform across the wave: held in a scalar register, the
  // per-wave weight and index addresses are scalar arithmetic
  const int tid0 = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid0 >> 6);
  const int64_t e0 = (int64_t)blockIdx.x * T;

  float logs = 0.0f;
#pragma unroll 1
  for (int k = 0; k < nl; ++k) {
    const int l = INVERSE ? nl - 1 - k : k;
    const LayerDev& L = layers.L[l];
    const int tid = fresh(tid0), lane = tid & 63, row = lane & 15, quad = lane >> 4;

    // inputs of the first dense layer (events fastest, so the reads coalesce):
    // each kept coordinate as a BF16 pair hi + lo (about 16 significant bits),
    // multiplied by the same weight column
    {
      // all of this thread's HBM reads are issued before the first is used
      // (one latency instead of several): kept coordinates w, w + 4, w + 8,
      // w + 12 and transformed coordinates w, w + 4 of event m (w = wave); the
      // transformed ones wait in LDS for their PQ transforms
      static_assert(KLO == 16 && TBMAX == 8, "four kept and two transformed coordinates per thread");
      const int m = lane;
      const int64_t e = e0 + m;
      const bool ev = e < n;
      float v[4], tv[2];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = wave + 4 * r;
        v[r] = (i < L.dA && ev) ? y[(int64_t)L.a_idx[i] * ld + e] : 0.0f;
      }
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int j = wave + 4 * r;
        tv[r] = (j < L.dB && ev) ? y[(int64_t)L.b_idx[j] * ld + e] : 0.5f;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = wave + 4 * r;
        const bf16 hi = (bf16)v[r];
        const bf16 lo = (bf16)(v[r] - (float)hi);
        const int il = i + KLO;
        xa[m * KA + (((i >> 3) ^ (m & 3)) << 3) + (i & 7)] = hi;
        xa[m * KA + (((il >> 3) ^ (m & 3)) << 3) + (il & 7)] = lo;
      }
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int j = wave + 4 * r;
        if (j < L.dB) tb[j * T + m] = tv[r];
      }
    }
    if (CACHE) {
      for (int idx = tid; idx < T * d; idx += 256) {
        const int m = idx % T, j = idx / T;
        const int64_t e = e0 + m;
        if (e < n) lin[l * lstride + (int64_t)j * n + e] = y[(int64_t)j * ld + e];
      }
    }
    __syncthreads();

    // Dense layers 1 and 2 are computed transposed, D[feature][event] =
    // W^T X^T: the weight rows are the A fragments (16-byte loads from the
    // [out][in] copies), the activations in LDS the B fragments, and each lane
    // ends with four consecutive features of one event, stored as one 8-byte
    // LDS write after bias and activation.  Wave w owns features [64w, 64w+64).
    {
      f32x4 acc[4][4];
      bf16x8 a[4], b[4];
#pragma unroll
      for (int jt = 0; jt < 4; ++jt)
        a[jt] = *reinterpret_cast<const bf16x8*>(L.W1t + (64 * wave + 16 * jt + row) * KA + 8 * quad);
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        const int m = 16 * mt + row;
        b[mt] = *reinterpret_cast<const bf16x8*>(xa + m * KA + ((quad ^ (m & 3)) << 3));
      }
#pragma unroll
      for (int jt = 0; jt < 4; ++jt) {
        const f32x4 bias = bias4(L.b1, wave, jt, quad);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) acc[jt][mt] = mfma16(a[jt], b[mt], bias);
      }
      store_features(h, acc, wave, row, quad);
    }
    __syncthreads();
    {
      f32x4 acc[4][4];
#pragma unroll
      for (int jt = 0; jt < 4; ++jt) {
        const f32x4 bias = bias4(L.b2, wave, jt, quad);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) acc[jt][mt] = bias;
      }
      // this wave's fragments in packed order: step ks, fragment jt at
      // ((wave 8 + ks) 4 + jt) KB; a step's fragments are requested two steps
      // ahead (a ring of three) and kept in their step by a scheduling barrier
      const bf16* W2 = L.W2p + (int64_t)wave * 8 * 4 * 512 + lane * 8;
      bf16x8 a[3][4];
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int jt = 0; jt < 4; ++jt) a[st][jt] = *reinterpret_cast<const bf16x8*>(W2 + (st * 4 + jt) * 512);
#pragma unroll
      for (int ks = 0; ks < H / 32; ++ks) {
        if (ks + 2 < H / 32) {
#pragma unroll
          for (int jt = 0; jt < 4; ++jt)
            a[(ks + 2) % 3][jt] = *reinterpret_cast<const bf16x8*>(W2 + ((ks + 2) * 4 + jt) * 512);
        }
        bf16x8 b[4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
          b[mt] = *reinterpret_cast<const bf16x8*>(h + hs(16 * mt + row, 32 * ks + 8 * quad));
#pragma unroll
        for (int jt = 0; jt < 4; ++jt)
#pragma unroll
          for (int mt = 0; mt < 4; ++mt) acc[jt][mt] = mfma16(a[ks % 3][jt], b[mt], acc[jt][mt]);
        __builtin_amdgcn_sched_barrier(0);
      }
      // every wave has read the first layer before the second overwrites it
      __syncthreads();
      store_features(h, acc, wave, row, quad);
    }
    __syncthreads();

    // The 65th logit of every transformed coordinate at once: one more MFMA
    // tile per wave, D[coordinate][event] for the wave's 16 events, with the
    // weight rows of the coordinates' last outputs as A fragments (packed;
    // rows past d_B are zero and never read).  Lane l keeps coordinates
    // 4 (l >> 4) + i of event 16 wave + (l & 15) in registers until their PQ
    // transforms.
    f32x4 lastv = {0.0f, 0.0f, 0.0f, 0.0f};
    {
      const bf16* wl = L.W3L + lane * 8;
#pragma unroll
      for (int ks = 0; ks < H / 32; ++ks) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(wl + ks * 512);
        const bf16x8 b = *reinterpret_cast<const bf16x8*>(h + hs(16 * wave + row, 32 * ks + 8 * quad));
        lastv = mfma16(a, b, lastv);
      }
    }

    // dense layer 3 and the PQ transform, one transformed coordinate at a time:
    // the 64 leading logits of a coordinate are four 16-column MFMA tiles, one
    // per wave over all 64 events (each wave streams only its own weight
    // columns).
    float lq = 0.0f;
    // the eight weight fragments of this wave's columns of coordinate c; those
    // of coordinate c + 1 are requested before the PQ transform of c, so their
    // L2 latency overlaps it
    bf16x8 bw[H / 32];
    {
      const bf16* W3 = L.W3p + (int64_t)wave * 8 * 512 + lane * 8;
#pragma unroll
      for (int ks = 0; ks < H / 32; ++ks) bw[ks] = *reinterpret_cast<const bf16x8*>(W3 + ks * 512);
    }
    // the PQ transform's event (16 per wave, four lanes each) and part
    const int m = tid >> 2, part = tid & 3;
    const int64_t em = e0 + m;
    const bool live = em < n;
    for (int c = 0; c < L.dB; ++c) {
      {
        const int col = 16 * wave + row;
        const float bias = L.b3p[c * NOP + col];
        f32x4 acc[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] = f32x4{bias, bias, bias, bias};
#pragma unroll
        for (int ks = 0; ks < H / 32; ++ks) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const bf16x8 a = *reinterpret_cast<const bf16x8*>(h + hs(16 * r + row, 32 * ks + 8 * quad));
            acc[r] = mfma16(a, bw[ks], acc[r]);
          }
        }
        if (c + 1 < L.dB) {
          const bf16* W3 = L.W3p + (((int64_t)(c + 1) * 4 + wave) * 8) * 512 + lane * 8;
#pragma unroll
          for (int ks = 0; ks < H / 32; ++ks) bw[ks] = *reinterpret_cast<const bf16x8*>(W3 + ks * 512);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int i = 0; i < 4; ++i) out[(16 * r + 4 * quad + i) * LDO + col] = acc[r][i];
      }
      // the 65th logit of (event m, coordinate c) from the lane of this wave
      // that holds it
      const int ci = c & 3;
      const float lsel = ci == 0 ? lastv[0] : ci == 1 ? lastv[1] : ci == 2 ? lastv[2] : lastv[3];
      const float vlast = __shfl(lsel, (lane >> 2) + 16 * (c >> 2)) + L.b3p[c * NOP + 2 * KB];
      __syncthreads();
      {
        float* yp = y + (int64_t)L.b_idx[c] * ld + (live ? em : e0);
        const float t = tb[c * T + m];
        float res, pdf;
        pq_quad<INVERSE>(out + m * LDO, vlast, t, part, res, pdf);
        if (live && part == 0) {
          *yp = res;
          lq += __logf(pdf);
        }
      }
      __syncthreads();
    }
    logs = k == 0 ? lq : logs + lq;
  }
  if ((tid0 & 3) == 0) {
    const int64_t e = e0 + (tid0 >> 2);
    if (e < n) logq[e] = logs;
  }
}

// -------------------------------------------------------- backward layer
// Operands of the weight gradients, event-major; those of the l-th layer held
// are l stride elements further.
struct Operands {
  bf16* xa;   // [n][KA]  inputs of the first dense layer (hi | lo)
  bf16* h1;   // [n][H]   hidden activations
  bf16* h2;   // [n][H]
  bf16* go;   // [n][dB*NOG] gradients of the logits (zero-padded per coordinate)
  bf16* ga2;  // [n][H]   gradients before the second activation
  bf16* ga1;  // [n][H]   and before the first
  int64_t stride;
};

// Sign bits of a lane's 64 features of a hidden layer, in the order of
// store_features: bit (jt 4 + mt) 4 + i.
struct Signs {
  unsigned b[2];
};
// store_features that also returns which rounded activations are positive.
__device__ __forceinline__ Signs store_features_signs(bf16* h, const f32x4 (&acc)[4][4], int wave, int row, int quad) {
  Signs s{{0u, 0u}};
#pragma unroll
  for (int jt = 0; jt < 4; ++jt) {
    const int f0 = 64 * wave + 16 * jt + 4 * quad;
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      bf16x4 v;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[i] = (bf16)leaky(acc[jt][mt][i]);
        s.b[jt >> 1] |= (float)v[i] > 0.0f ? 1u << ((jt & 1) * 16 + mt * 4 + i) : 0u;
      }
      *reinterpret_cast<bf16x4*>(h + hs(16 * mt + row, f0)) = v;
    }
  }
  // the bits now, not the activations until the bits are used
  asm volatile("" : "+v"(s.b[0]), "+v"(s.b[1]));
  return s;
}
// The gradient before an activation from the one after it, rounded to BF16
// and stored as store_features does.
__device__ __forceinline__ void store_gradients(bf16* h, const f32x4 (&acc)[4][4], Signs s, int wave, int row, int quad) {
#pragma unroll
  for (int jt = 0; jt < 4; ++jt) {
    const int f0 = 64 * wave + 16 * jt + 4 * quad;
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      bf16x4 v;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        v[i] = (bf16)(acc[jt][mt][i] * ((s.b[jt >> 1] >> ((jt & 1) * 16 + mt * 4 + i)) & 1u ? 1.0f : SLOPE));
      *reinterpret_cast<bf16x4*>(h + hs(16 * mt + row, f0)) = v;
    }
  }
}
// The [T][H] tile to rows e0.. of an event-major matrix: 512 consecutive
// bytes per event, past the caches.
__device__ __forceinline__ void copy_tile(const bf16* h, bf16* __restrict__ dst, int64_t e0, int64_t n, int tid) {
#pragma unroll
  for (int r = 0; r < T * H / 8 / 256; ++r) {
    const int idx = tid + 256 * r, m = idx >> 5, k = 8 * (idx & 31);
    if (e0 + m < n)
      __builtin_nontemporal_store(*reinterpret_cast<const bf16x8*>(h + hs(m, k)),
                                  reinterpret_cast<bf16x8*>(dst + (e0 + m) * H + k));
  }
}
// Logit-gradient tile of one coordinate: [T][64] bf16, the eight 16-byte
// chunks of a row permuted so that the 16 rows of a fragment load fall in
// different banks.
__device__ __forceinline__ int gs(int m, int chunk) { return m * 64 + ((chunk ^ ((m ^ (m >> 3)) & 7)) << 3); }
// After it, a chunk per event for the last logit of an even and of an odd
// coordinate (the other seven elements stay zero), and one chunk of zeros.
__device__ __forceinline__ int gs_last(int m, int odd) { return T * 64 + (odd * T + m) * 8; }
constexpr int GS_ZERO = T * 64 + 2 * T * 8;
constexpr int GT_CHUNKS = GS_ZERO / 8 + 1;

// Value of lane S of each aligned group of four.
template <int S> __device__ __forceinline__ float qlane(float x) { return qdpp<0x55 * S>(x); }
// Sum over the four lanes' terms in order (lane 0's first), each lane adding
// its terms one by one with f(running sum); every lane returns the total,
// and start receives the sum before this lane's terms.
template <class F> __device__ __forceinline__ float ordered_sum(int p, float& start, F f) {
  float t = 0.0f;
  start = 0.0f;
  t = qlane<0>(f(t));
  start = p == 1 ? t : start;
  t = qlane<1>(f(t));
  start = p == 2 ? t : start;
  t = qlane<2>(f(t));
  start = p == 3 ? t : start;
  return qlane<3>(f(t));
}

// Derivatives of the PQ transform of one coordinate (density direction), four
// lanes per event as in pq_quad, lane part p holding bins and vertices
// [8p, 8p+8): from the gradient gz of the loss with respect to the
// transform's output and glp with respect to its log density, the gradients
// gw[k] and gv[k] of the part's width and vertex logits, glast of the last
// vertex logit (p = 3), and the gradient with respect to the input yv.  Sums
// over bins run in bin order, and the products that are added use one rounding.
__device__ __forceinline__ void pq_quad_backward(const float* o, float vlast, float yv, int p, float gz, float glp,
                                                 float (&gw)[KB / 4], float (&gv)[KB / 4], float& glast, float& gy) {
  constexpr int KP = KB / 4;
  float W[KP], V[KP + 1], start;
#pragma unroll
  for (int k = 0; k < KP; ++k) W[k] = o[KP * p + k];
#pragma unroll
  for (int k = 0; k < KP; ++k) V[k] = o[KB + KP * p + k];
  {
    const float vn = o[KB + KP * p + (p < 3 ? KP : 0)];
    V[KP] = p < 3 ? vn : vlast;
  }
  float mw = W[0];
#pragma unroll
  for (int k = 1; k < KP; ++k) mw = fmaxf(mw, W[k]);
  mw = max_nc(mw, qdpp<QX1>(mw));
  mw = max_nc(mw, qdpp<QX2>(mw));
#pragma unroll
  for (int k = 0; k < KP; ++k) W[k] = __expf(W[k] - mw);
  const float sw = ordered_sum(p, start, [&](float t) {
#pragma unroll
    for (int k = 0; k < KP; ++k) t += W[k];
    return t;
  });
  const float isw = 1.0f / sw;
  // bin b of the point: the largest k >= 1 whose left edge is <= yv, else 0;
  // the edges are running sums of the widths, each product and sum one rounding
  (void)ordered_sum(p, start, [&](float t) {
#pragma unroll
    for (int k = 0; k < KP; ++k) t = __builtin_fmaf(W[k], isw, t);
    return t;
  });
  int b = p == 0 || start <= yv ? KP * p : -1;
  float S = start, Sb = S, first2 = 0.0f;
#pragma unroll
  for (int k = 0; k < KP; ++k) {
    const bool take = k > 0 && S <= yv;
    b = take ? KP * p + k : b;
    Sb = take ? S : Sb;
    S = __builtin_fmaf(W[k], isw, S);
    if (k == 1) first2 = S;
  }
  b = max(b, qdpp<QX1>(b));
  b = max(b, qdpp<QX2>(b));
#pragma unroll
  for (int k = 0; k < KP; ++k) W[k] *= isw;
  float mv = V[0];
#pragma unroll
  for (int k = 1; k <= KP; ++k) mv = fmaxf(mv, V[k]);
  mv = max_nc(mv, qdpp<QX1>(mv));
  mv = max_nc(mv, qdpp<QX2>(mv));
#pragma unroll
  for (int k = 0; k <= KP; ++k) V[k] = __expf(V[k] - mv);
  const float N = ordered_sum(p, start, [&](float t) {
#pragma unroll
    for (int k = 0; k < KP; ++k) t = __builtin_fmaf(0.5f * (V[k] + V[k + 1]), W[k], t);
    return t;
  });
  const float iN = 1.0f / N;
#pragma unroll
  for (int k = 0; k <= KP; ++k) V[k] *= iN;
  float Wb = W[0], Vb = V[0], Vb1 = V[1];
#pragma unroll
  for (int k = 1; k < KP; ++k) {
    const bool at = KP * p + k == b;
    Wb = at ? W[k] : Wb;
    Vb = at ? V[k] : Vb;
    Vb1 = at ? V[k + 1] : Vb1;
  }
  {
    const bool own = (b >> 3) == p;
    auto bcast = [&](float v) {
      float x = own ? v : 0.0f;
      x += qdpp<QX1>(x);
      return x + qdpp<QX2>(x);
    };
    Sb = bcast(Sb);
    Wb = bcast(Wb);
    Vb = bcast(Vb);
    Vb1 = bcast(Vb1);
  }
  const float al = fminf(fmaxf((yv - Sb) / Wb, 0.0f), 1.0f);
  const float dV = Vb1 - Vb;
  const float pdf = __builtin_fmaf(al, dV, Vb);
  const float gp = glp / pdf, slope = dV / Wb;
  // d/dW_k and d/dV_k of (gz z + glp log pdf) at fixed logits of other bins
  const float wl0 = qdpp<0x90>(W[KP - 1]);  // the width before the part's first (lane p - 1)
  const float vat = __builtin_fmaf(gz * Wb, __builtin_fmaf(al, -0.5f * al, al), gp * (1.0f - al));
  const float vnext = __builtin_fmaf(gz * Wb * 0.5f * al, al, gp * al);
#pragma unroll
  for (int k = 0; k < KP; ++k) {
    const int kk = KP * p + k;
    const bool below = kk < b, at = kk == b;
    const float dz = below ? __builtin_fmaf(-al, dV, __builtin_fmaf(0.5f, V[k] + V[k + 1], -Vb))
                           : (at ? -0.5f * al * al * dV : 0.0f);
    const float dp = below ? -slope : (at ? -al * dV / Wb : 0.0f);
    gw[k] = __builtin_fmaf(gz, dz, gp * dp);
    // area terms of z: A_b = sum_{k<b} W_k (V_k + V_k+1)/2
    const float wl = k > 0 ? W[k - 1] : wl0;
    float g = kk >= 1 && kk - 1 < b ? gz * 0.5f * wl : 0.0f;
    g = below ? __builtin_fmaf(gz * 0.5f, W[k], g) : g;
    g += at ? vat : 0.0f;
    g += kk == b + 1 ? vnext : 0.0f;
    gv[k] = g;
  }
  glast = KB - 1 < b ? gz * 0.5f * W[KP - 1] : 0.0f;
  glast += b + 1 == KB ? vnext : 0.0f;
  gy = __builtin_fmaf(gz, pdf, glp * slope / pdf);
  // through V = exp(v) / N, N = sum_k W_k (exp(v_k) + exp(v_k+1)) / 2, and W = softmax
  const float sg = ordered_sum(p, start, [&](float t) {
#pragma unroll
    for (int k = 0; k < KP; ++k) t = __builtin_fmaf(gv[k], V[k], t);
    return t;
  });
  const float SG = qlane<3>(__builtin_fmaf(glast, V[KP], sg));
#pragma unroll
  for (int k = 0; k < KP; ++k) gw[k] = __builtin_fmaf(-(V[k] + V[k + 1]), SG * 0.5f, gw[k]);
  const float SW = ordered_sum(p, start, [&](float t) {
#pragma unroll
    for (int k = 0; k < KP; ++k) t = __builtin_fmaf(W[k], gw[k], t);
    return t;
  });
#pragma unroll
  for (int k = 0; k < KP; ++k) {
    gw[k] = W[k] * (gw[k] - SW);
    const float wl = k > 0 ? W[k - 1] : (p > 0 ? wl0 : 0.0f);
    // the first two widths together are the second edge
    const float ws = k == 1 && p == 0 ? first2 : wl + W[k];
    gv[k] = V[k] * __builtin_fmaf(-ws, SG * 0.5f, gv[k]);
  }
  glast = V[KP] * __builtin_fmaf(-W[KP - 1], SG * 0.5f, glast);
}

// The backward pass through layers l1 - 1 .. l0 of nl (all of them where their
// operands fit) for events [64 blockIdx.x, +64); as in the forward pass a tile
// needs no other.  Of each layer, the last first,
// the hidden layers and the logits are computed again from the layer's input
// lin + l lstride ([d][n]; the same products as in k_coupling, cheaper than
// keeping 2.4 KB per event and layer), each coordinate's logits give the
// gradients of its PQ transform, which are multiplied into the gradient of the
// second hidden layer at once, and so on to the kept inputs.  g ([d][n]) holds
// the gradient with respect to the current layer's output, zero at the last,
// and receives the one with respect to its input; glp = dL/dlog q =
// -w_e / sum w.  Written besides: the operands of the weight gradients, in rows
// of 64 to 1152 bytes per event.  The products run transposed,
// D[feature][event], so that a lane's gradients are the features whose
// activations it computed and their signs stay in two registers per layer.
//
// LDS: the [T][H] tile holds the first hidden layer, the second, the gradient
// before the second activation and that before the first; the logits of the
// current coordinate (before that, the first layer's inputs); its logit
// gradients; the transformed inputs: 61 KiB, two workgroups per compute unit.
//
// Sums over bins, and over k in the products, keep one fixed order: a BF16
// rounding that falls the other way changes an event's gradient by 2^-9.
//
// The operands are stored past the caches: they are read by the next launch
// only, 1.1 GB for 65536 points of 10 dimensions, and would push the weights
// of six layers (4.5 MB) out of the L2 (735 us, with these stores 590).
//
// 65536 points of 10 dimensions, six layers: 577 us at two waves per SIMD.
// Vector instructions other than the matrix ones are issued in 43 % of the SIMD
// cycles, the matrix cores are busy in 19 %, and a wave waits half of its time.
// As separate kernels over cached activations and logits the same work took 285
// us per layer: PQ derivatives 67, two products with BF16 epilogues 76 each, the
// input product 17, its addition 6, and 43 for writing the caches in the forward
// pass.
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
k_backward(Layers layers, int nl, int l0, int l1, const float* __restrict__ lin_all, int64_t lstride, int64_t n, float* __restrict__ g,
           const float* __restrict__ w, const float* __restrict__ wsum, Operands op, int d) {
  __shared__ __attribute__((aligned(16))) bf16 h[T * H];
  __shared__ __attribute__((aligned(16))) float out[T * LDO];
  __shared__ __attribute__((aligned(16))) bf16 gt[GT_CHUNKS * 8];
  __shared__ float tb[TBMAX * T];
  bf16* xa = reinterpret_cast<bf16*>(out);  // [T][KA]
  const int tid0 = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid0 >> 6);
  const int64_t e0 = (int64_t)blockIdx.x * T;
  for (int idx = l1 == nl ? tid0 : T * d; idx < T * d; idx += 256)
    if (e0 + idx % T < n) g[(int64_t)(idx / T) * n + e0 + idx % T] = 0.0f;
#pragma unroll 1
  for (int l = l1 - 1; l >= l0; --l) {
    const LayerDev& L = layers.L[l];
    const float* lin = lin_all + l * lstride;
    Operands out_op = op;
    out_op.xa += (l - l0) * op.stride;
    out_op.h1 += (l - l0) * op.stride;
    out_op.h2 += (l - l0) * op.stride;
    out_op.go += (l - l0) * op.stride;
    out_op.ga2 += (l - l0) * op.stride;
    out_op.ga1 += (l - l0) * op.stride;
    const int tid = fresh(tid0), lane = tid & 63, row = lane & 15, quad = lane >> 4;
    // inputs as in k_coupling
    {
      const int m = lane;
      const int64_t e = e0 + m;
      const bool ev = e < n;
      float v[4], tv[2];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = wave + 4 * r;
        v[r] = (i < L.dA && ev) ? lin[(int64_t)L.a_idx[i] * n + e] : 0.0f;
      }
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int j = wave + 4 * r;
        tv[r] = (j < L.dB && ev) ? lin[(int64_t)L.b_idx[j] * n + e] : 0.5f;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = wave + 4 * r;
        const bf16 hi = (bf16)v[r];
        const bf16 lo = (bf16)(v[r] - (float)hi);
        const int il = i + KLO;
        xa[m * KA + (((i >> 3) ^ (m & 3)) << 3) + (i & 7)] = hi;
        xa[m * KA + (((il >> 3) ^ (m & 3)) << 3) + (il & 7)] = lo;
      }
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int j = wave + 4 * r;
        if (j < L.dB) tb[j * T + m] = tv[r];
      }
      for (int i = T * 64 + tid; i < GT_CHUNKS * 8; i += 256) gt[i] = (bf16)0.0f;
    }
    __syncthreads();
    {
      const int m = tid >> 2, k = tid & 3;  // one 16-byte chunk of the inputs per thread
      if (e0 + m < n)
        *reinterpret_cast<bf16x8*>(out_op.xa + (e0 + m) * KA + 8 * k) =
            *reinterpret_cast<const bf16x8*>(xa + m * KA + ((k ^ (m & 3)) << 3));
    }
    Signs s1, s2;
    {
      f32x4 acc[4][4];
      bf16x8 a[4], b[4];
#pragma unroll
      for (int jt = 0; jt < 4; ++jt)
        a[jt] = *reinterpret_cast<const bf16x8*>(L.W1t + (64 * wave + 16 * jt + row) * KA + 8 * quad);
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        const int m = 16 * mt + row;
        b[mt] = *reinterpret_cast<const bf16x8*>(xa + m * KA + ((quad ^ (m & 3)) << 3));
      }
#pragma unroll
      for (int jt = 0; jt < 4; ++jt) {
        const f32x4 bias = bias4(L.b1, wave, jt, quad);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) acc[jt][mt] = mfma16(a[jt], b[mt], bias);
      }
      s1 = store_features_signs(h, acc, wave, fresh(row), quad);
    }
    __syncthreads();
    copy_tile(h, out_op.h1, e0, n, fresh(tid));
    // [H x H] product with the tile: fragments of packed rows W, as in k_coupling
    auto dense = [&](const bf16* Wp, f32x4 (&acc)[4][4]) {
      const bf16* W2 = Wp + (int64_t)wave * 8 * 4 * 512 + lane * 8;
      const int rb = fresh(row);
      bf16x8 a[3][4];
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int jt = 0; jt < 4; ++jt) a[st][jt] = *reinterpret_cast<const bf16x8*>(W2 + (st * 4 + jt) * 512);
#pragma unroll
      for (int ks = 0; ks < H / 32; ++ks) {
        if (ks + 2 < H / 32) {
#pragma unroll
          for (int jt = 0; jt < 4; ++jt)
            a[(ks + 2) % 3][jt] = *reinterpret_cast<const bf16x8*>(W2 + ((ks + 2) * 4 + jt) * 512);
        }
        bf16x8 b[4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
          b[mt] = *reinterpret_cast<const bf16x8*>(h + hs(16 * mt + rb, 32 * ks + 8 * quad));
#pragma unroll
        for (int jt = 0; jt < 4; ++jt)
#pragma unroll
          for (int mt = 0; mt < 4; ++mt) acc[jt][mt] = mfma16(a[ks % 3][jt], b[mt], acc[jt][mt]);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    {
      f32x4 acc[4][4];
#pragma unroll
      for (int jt = 0; jt < 4; ++jt) {
        const f32x4 bias = bias4(L.b2, wave, jt, quad);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) acc[jt][mt] = bias;
      }
      dense(L.W2p, acc);
      __syncthreads();  // every wave has read the first layer
      s2 = store_features_signs(h, acc, wave, fresh(row), quad);
    }
    __syncthreads();
    copy_tile(h, out_op.h2, e0, n, fresh(tid));
    f32x4 lastv = {0.0f, 0.0f, 0.0f, 0.0f};
    {
      const bf16* wl = L.W3L + lane * 8;
#pragma unroll
      for (int ks = 0; ks < H / 32; ++ks) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(wl + ks * 512);
        const bf16x8 b = *reinterpret_cast<const bf16x8*>(h + hs(16 * wave + row, 32 * ks + 8 * quad));
        lastv = mfma16(a, b, lastv);
      }
    }
    // gradient after the second activation, accumulated over the coordinates
    f32x4 acc[4][4];
#pragma unroll
    for (int jt = 0; jt < 4; ++jt)
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) acc[jt][mt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const int m = tid >> 2, part = tid & 3;
    const int64_t em = e0 + m;
    const bool live = em < n;
    const float glp = live ? -w[em] / wsum[0] : 0.0f;
    const int NB = L.dB * NOG;
    for (int c = 0; c < L.dB; ++c) {
      {
        const bf16* W3 = L.W3p + (((int64_t)c * 4 + wave) * 8) * 512 + lane * 8;
        const int col = 16 * wave + row;
        const float bias = L.b3p[c * NOP + col];
        f32x4 lg[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) lg[r] = f32x4{bias, bias, bias, bias};
#pragma unroll
        for (int ks = 0; ks < H / 32; ++ks) {
          const bf16x8 bw = *reinterpret_cast<const bf16x8*>(W3 + ks * 512);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const bf16x8 a = *reinterpret_cast<const bf16x8*>(h + hs(16 * r + row, 32 * ks + 8 * quad));
            lg[r] = mfma16(a, bw, lg[r]);
          }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int i = 0; i < 4; ++i) out[(16 * r + 4 * quad + i) * LDO + col] = lg[r][i];
      }
      const int ci = c & 3;
      const float lsel = ci == 0 ? lastv[0] : ci == 1 ? lastv[1] : ci == 2 ? lastv[2] : lastv[3];
      const float vlast = __shfl(lsel, (lane >> 2) + 16 * (c >> 2)) + L.b3p[c * NOP + 2 * KB];
      float* gp = g + (int64_t)L.b_idx[c] * n + (live ? em : e0);
      const float gz = live ? *gp : 0.0f;
      // this coordinate's fragments for the gradient, requested before the PQ
      // derivatives
      const int odd = c & 1;
      const bf16* wqc = L.W3q + ((int64_t)((c >> 1) * 5 + 2 * odd) * 16 + wave * 4) * 512 + lane * 8;
      bf16x8 wq[2][4];
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int jt = 0; jt < 4; ++jt) wq[st][jt] = *reinterpret_cast<const bf16x8*>(wqc + (st * 16 + jt) * 512);
      __syncthreads();  // logits complete; the previous coordinate's gradients have been read
      {
        float gw[KB / 4], gv[KB / 4], gl, gy;
        pq_quad_backward(out + m * LDO, vlast, tb[c * T + m], part, gz, glp, gw, gv, gl, gy);
        if (live && part == 0) *gp = gy;
        bf16x8 a, b;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          a[k] = (bf16)gw[k];
          b[k] = (bf16)gv[k];
        }
        bf16x8 l8;
#pragma unroll
        for (int k = 0; k < 8; ++k) l8[k] = k == 0 ? (bf16)gl : (bf16)0.0f;
        *reinterpret_cast<bf16x8*>(gt + gs(m, part)) = a;
        *reinterpret_cast<bf16x8*>(gt + gs(m, 4 + part)) = b;
        if (part == 3) gt[gs_last(m, odd)] = (bf16)gl;
        if (live) {
          bf16* dst = out_op.go + em * NB + c * NOG;
          __builtin_nontemporal_store(a, reinterpret_cast<bf16x8*>(dst + 8 * part));
          __builtin_nontemporal_store(b, reinterpret_cast<bf16x8*>(dst + KB + 8 * part));
          if (part == 3) __builtin_nontemporal_store(l8, reinterpret_cast<bf16x8*>(dst + 2 * KB));
        }
      }
      __syncthreads();
      // k steps of 32 over NOP columns per coordinate: two for an even
      // coordinate; three for an odd one, the first beginning with the last
      // logit of the one before, the third ending with its own.  An even last
      // coordinate ends with a step of its last logit.
      auto step = [&](const bf16x8 (&aw)[4], int chunk) {
        bf16x8 b[4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
          const int mm = 16 * mt + row;
          int at = gs(mm, chunk & 7);
          at = chunk < 0 || chunk > 8 ? GS_ZERO : at;
          at = chunk == -2 || chunk == 8 ? gs_last(mm, chunk == 8 ? odd : 0) : at;
          b[mt] = *reinterpret_cast<const bf16x8*>(gt + at);
        }
#pragma unroll
        for (int jt = 0; jt < 4; ++jt)
#pragma unroll
          for (int mt = 0; mt < 4; ++mt) acc[jt][mt] = mfma16(aw[jt], b[mt], acc[jt][mt]);
      };
      step(wq[0], quad - 2 * odd);
      step(wq[1], quad + 4 - 2 * odd);
      if (odd || c + 1 == L.dB) {
#pragma unroll
        for (int jt = 0; jt < 4; ++jt) wq[0][jt] = *reinterpret_cast<const bf16x8*>(wqc + (32 + jt) * 512);
        step(wq[0], quad + 8 - 2 * odd);
      }
    }
    // every wave read the second layer before the barriers of the last coordinate
    store_gradients(h, acc, s2, wave, fresh(row), quad);
    __syncthreads();
    copy_tile(h, out_op.ga2, e0, n, fresh(tid));
#pragma unroll
    for (int jt = 0; jt < 4; ++jt)
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) acc[jt][mt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    dense(L.W2q, acc);
    __syncthreads();
    store_gradients(h, acc, s1, wave, fresh(row), quad);
    __syncthreads();
    copy_tile(h, out_op.ga1, e0, n, fresh(tid));
    // gradient reaching the kept coordinates: D[coordinate][event], the wave's
    // 16 events
    f32x4 gx = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int ks = 0; ks < H / 32; ++ks) {
      const bf16x8 a = *reinterpret_cast<const bf16x8*>(L.W1q + ks * 512 + lane * 8);
      const bf16x8 b = *reinterpret_cast<const bf16x8*>(h + hs(16 * wave + row, 32 * ks + 8 * quad));
      gx = mfma16(a, b, gx);
    }
    const int64_t eg = e0 + 16 * wave + row;
    if (eg < n) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int ci = 4 * quad + i;
        if (ci < L.dA) g[(int64_t)L.a_idx[ci] * n + eg] += gx[i];
      }
    }
    __syncthreads();  // the layer's gradients are written and its tiles read
  }
}

// ------------------------------------------------------ weight gradients
// dW[m][j] = sum over events of X[e][m] G[e][j] for the three dense layers of
// every coupling layer (X = h2, h1, xa and G = go, ga2, ga1), with the column
// sums of G (the bias gradients) as row M, in partials over chunks of events:
// part[z zs + off + m N + j].  All products are one launch, numbered so that the
// tiles of one chunk run on one XCD, those of one layer together, and share
// their operands in its L2.  A workgroup takes a 128 x 128 tile, each of its
// four waves 64 x 64: a fragment read from LDS then serves four matrix
// instructions (two for the 32 x 32 of a 64 x 64 tile, which is bound by LDS
// reads).  The operands are event-major and the events are the contraction, so
// the fragments come from LDS transposed (ds_read_b64_tr_b16): a group of 16
// lanes reads 4 events x 16 features, lane i receiving feature i of the four
// events.  Per k step of 32 events lane group q takes events 4q..4q+3 and
// 16+4q..16+4q+3 for both operands; with rows of 288 bytes the 8 rows of half a
// wave fall in different banks (no conflicts counted).  Bound by memory: six
// layers of 65536 points of 10 dimensions have 1.1 GB of operands, read 1.5
// times: 284 us (6.0 TB/s), and 11 us for the reduction.  Launched layer by layer beside
// the backward pass, with six times the partials, the whole gradient took 1.42
// ms instead of 1.11; three launches per layer of 64 x 64 tiles on
// event-contiguous copies and three reductions took 250 us per layer.
constexpr int WT = 128;        // tile edge
constexpr int WK = 64;         // events per staged slice: two k steps
constexpr int WLD = WT + 16;   // LDS row stride (bf16)
struct Product {
  const bf16* X;
  const bf16* G;
  int M, N;
  int tiles_n, first;  // column tiles; first tile number
  int64_t off;         // of its partials
};
struct WgradArgs {
  Product p[3 * MAXL];
  int np, tiles;  // products and their tiles
  int64_t zs;     // floats of one chunk's partials
  int64_t n, chunk;
  int64_t zmax;   // chunks at most, of n events or fewer
  float* part;
};
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bf16x8 tr_fragment(const bf16* base, int k, int f, int lane) {
  // events k + 4q + (0..3) and k + 16 + 4q + (0..3), feature f + (lane & 15)
  typedef __attribute__((address_space(3))) s16x4* P;
  const int q = lane >> 4, i = lane & 15;
  const bf16* p = base + (k + 4 * q + (i >> 2)) * WLD + f + 4 * (i & 3);
  union {
    s16x4 s[2];
    bf16x8 v;
  } u;
  u.s[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((P)p);
  u.s[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((P)(p + 16 * WLD));
  return u.v;
}
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) k_wgrad(WgradArgs a) {
  __shared__ __attribute__((aligned(16))) bf16 Xs[2][WK * WLD];
  __shared__ __attribute__((aligned(16))) bf16 Gs[2][WK * WLD];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row = lane & 15, quad = lane >> 4;
  // workgroup b runs on XCD b mod 8: tiles are numbered XCD by XCD
  const int G = gridDim.x, xcd = blockIdx.x & 7, per = G >> 3, rem = G & 7;
  const int t = xcd * per + (xcd < rem ? xcd : rem) + (int)(blockIdx.x >> 3);
  const int z = t / a.tiles, tl = t % a.tiles;
  int pr = 0;
  for (int i = 1; i < a.np; ++i) pr = tl >= a.p[i].first ? i : pr;
  const Product& D = a.p[pr];
  const bf16* X = D.X;
  const bf16* Gp = D.G;
  const int M = D.M, N = D.N, tp = tl - D.first;
  const int m0 = tp / D.tiles_n * WT, n0 = tp % D.tiles_n * WT;
  const int64_t kb = (int64_t)z * a.chunk, ke = kb + a.chunk < a.n ? kb + a.chunk : a.n;
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
  f32x4 acc[4][4], accs[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    accs[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  const bool sums = m0 == 0 && wm == 0;
  const bool work = m0 + wm < M;  // the wave's rows exist (the first layer has 32)
  bf16x8 ones, zero;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    ones[i] = (bf16)1.0f;
    zero[i] = (bf16)0.0f;
  }
  // this thread's share of a slice: rows r0 + 16 r, eight features from c8;
  // rows past the chunk and columns past the matrix are loaded from an
  // in-range place and stored as zeros (M and N are multiples of 8)
  const int r0 = tid >> 4, c8 = (tid & 15) * 8;
  const bool vx = m0 + c8 < M, vg = n0 + c8 < N;
  const bf16* Xc = X + (vx ? m0 + c8 : 0);
  const bf16* Gc = Gp + (vg ? n0 + c8 : 0);
  // two register stages: the slices k + 1 and k + 2 are in flight while slice
  // k is multiplied
  bf16x8 rx[2][4], rg[2][4];
  auto load = [&](int64_t k0, bf16x8 (&x)[4], bf16x8 (&g)[4]) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t e = k0 + r0 + 16 * r, ec = e < ke ? e : kb;
      x[r] = *reinterpret_cast<const bf16x8*>(Xc + ec * M);
      g[r] = *reinterpret_cast<const bf16x8*>(Gc + ec * N);
    }
  };
  auto store = [&](int buf, int64_t k0, const bf16x8 (&x)[4], const bf16x8 (&g)[4]) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool ok = k0 + r0 + 16 * r < ke;
      *reinterpret_cast<bf16x8*>(&Xs[buf][(r0 + 16 * r) * WLD + c8]) = ok && vx ? x[r] : zero;
      *reinterpret_cast<bf16x8*>(&Gs[buf][(r0 + 16 * r) * WLD + c8]) = ok && vg ? g[r] : zero;
    }
  };
  auto products = [&](int buf) {
    if (!work) return;
#pragma unroll
    for (int kk = 0; kk < WK; kk += 32) {
      bf16x8 x[4], y[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = tr_fragment(Xs[buf], kk, wm + 16 * i, lane);
#pragma unroll
      for (int j = 0; j < 4; ++j) y[j] = tr_fragment(Gs[buf], kk, wn + 16 * j, lane);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = mfma16(x[i], y[j], acc[i][j]);
      if (sums) {
#pragma unroll
        for (int j = 0; j < 4; ++j) accs[j] = mfma16(ones, y[j], accs[j]);
      }
    }
  };
  // slice k is stored to buffer k mod 2, which was last read two slices
  // before, ahead of the previous slice's barrier; loads past the chunk read
  // its first event
  load(kb, rx[0], rg[0]);
  load(kb + WK, rx[1], rg[1]);
  int64_t k0 = kb;
  for (; k0 + WK < ke; k0 += 2 * WK) {
    store(0, k0, rx[0], rg[0]);
    __syncthreads();
    load(k0 + 2 * WK, rx[0], rg[0]);
    products(0);
    store(1, k0 + WK, rx[1], rg[1]);
    __syncthreads();
    load(k0 + 3 * WK, rx[1], rg[1]);
    products(1);
  }
  if (k0 < ke) {
    store(0, k0, rx[0], rg[0]);
    __syncthreads();
    products(0);
  }
  float* P = a.part + (int64_t)z * a.zs + D.off;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int gn = n0 + wn + 16 * j + row;
    if (gn >= N) continue;
    if (sums && quad == 0) P[(int64_t)M * N + gn] = accs[j][0];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int gm = m0 + wm + 16 * i + 4 * quad;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (gm + r < M) P[(int64_t)(gm + r) * N + gn] = acc[i][j][r];
    }
  }
}

// The gradients of layer blockIdx.y from the partials, summed over the chunks
// in order: W3 and b3 without the padding of each coordinate's columns, W2 and
// b2, W1 (the sum of the products with the high and the low input parts) and
// b1.
struct ReduceArgs {
  int dA[MAXL], dB[MAXL];
  int64_t off[MAXL], goff[MAXL];  // of the layer's partials and of its gradient
};
__global__ void __launch_bounds__(256) k_reduce_grad(const float* __restrict__ part_all, int Z, int64_t zs, ReduceArgs a,
                                                     float* __restrict__ grad_all) {
  const int dA = a.dA[blockIdx.y], dB = a.dB[blockIdx.y];
  const float* part = part_all + a.off[blockIdx.y];
  float* grad = grad_all + a.goff[blockIdx.y];
  const int N3 = dB * NOG, nO = dB * NO;
  const int64_t n3 = (int64_t)(H + 1) * N3, n2 = (int64_t)(H + 1) * H, n1 = (int64_t)(dA + 1) * H;
  int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n3 + n2 + n1) return;
  float* gW1 = grad;
  float* gb1 = gW1 + (int64_t)dA * H;
  float* gW2 = gb1 + H;
  float* gb2 = gW2 + (int64_t)H * H;
  float* gW3 = gb2 + H;
  const float* p = part + i;
  const float* q = nullptr;
  float* dst;
  if (i < n3) {
    const int m = (int)(i / N3), j = (int)(i % N3), c = j / NOG, r = j % NOG;
    if (r >= NO) return;
    dst = gW3 + (int64_t)m * nO + c * NO + r;  // row H: the bias gradients follow the weights
  } else if (i < n3 + n2) {
    dst = gW2 + (i - n3);
  } else {
    // rows 0..dA-1 and KLO.. of the KA input rows, and the sums in row KA
    i -= n3 + n2;
    const int m = (int)(i / H), j = (int)(i % H);
    p = part + n3 + n2 + (int64_t)(m < dA ? m : KA) * H + j;
    q = m < dA ? p + (int64_t)KLO * H : nullptr;
    dst = gW1 + i;
  }
  float s = 0.0f;
  if (q) {
    for (int z = 0; z < Z; ++z) {
      s += p[z * zs];
      s += q[z * zs];
    }
  } else {
#pragma unroll 8
    for (int z = 0; z < Z; ++z) s += p[z * zs];
  }
  *dst = s;
}

// sum of w over the batch (one block, fixed order) and the loss
// -sum w logq / sum w
constexpr int RB = 1024;  // threads of the single-block batch reductions
__global__ void __launch_bounds__(RB) k_wsum(const float* __restrict__ w, int64_t n, float* __restrict__ out) {
  __shared__ double s[RB];
  double a = 0.0;
#pragma unroll 8
  for (int64_t i = threadIdx.x; i < n; i += RB) a += w[i];
  s[threadIdx.x] = a;
  __syncthreads();
  for (int st = RB / 2; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) s[threadIdx.x] += s[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = (float)s[0];
}
// variance loss: per-point weights w^2 / q (held fixed in the backward pass)
__global__ void k_variance_weights(const float* __restrict__ w, const float* __restrict__ logq, int64_t n,
                                   float* __restrict__ weff) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n) weff[e] = w[e] * w[e] * __expf(-logq[e]);
}
// relative variance per event of sampling q, from points uniform in y:
// n sum w^2/q / (sum w)^2 - 1; and the sum of the weights w^2/q, as k_wsum
__global__ void __launch_bounds__(RB) k_relvar(const float* __restrict__ w, const float* __restrict__ weff, int64_t n,
                                               float* __restrict__ out, float* __restrict__ wsum) {
  __shared__ double s1[RB], s2[RB];
  double a = 0.0, b = 0.0;
#pragma unroll 8
  for (int64_t i = threadIdx.x; i < n; i += RB) {
    a += w[i];
    b += weff[i];
  }
  s1[threadIdx.x] = a;
  s2[threadIdx.x] = b;
  __syncthreads();
  for (int st = RB / 2; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) {
      s1[threadIdx.x] += s1[threadIdx.x + st];
      s2[threadIdx.x] += s2[threadIdx.x + st];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[0] = (float)((double)n * s2[0] / (s1[0] * s1[0]) - 1.0);
    wsum[0] = (float)s2[0];
  }
}
__global__ void __launch_bounds__(RB) k_loss(const float* __restrict__ w, const float* __restrict__ logq, int64_t n,
                                             const float* __restrict__ wsum, float* __restrict__ out) {
  __shared__ double s[RB];
  double a = 0.0;
#pragma unroll 8
  for (int64_t i = threadIdx.x; i < n; i += RB) a += (double)w[i] * logq[i];
  s[threadIdx.x] = a;
  __syncthreads();
  for (int st = RB / 2; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) s[threadIdx.x] += s[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = (float)(-s[0] / wsum[0]);
}

// Parameter segments of one layer in the master layout and the BF16 copies.
struct SegLayer {
  int64_t off;  // start of the layer in the master array
  int dA, dB;
  bf16* W1t;
  float* b3p;
  bf16* W2p;
  bf16* W3p;
  bf16* W3L;
  bf16* W2q;
  bf16* W3q;
  bf16* W1q;
};
struct SegTable {
  int nl;
  SegLayer l[MAXL];
};

// Adam on the masters (in place) and refresh of the BF16 copies.  With
// do_adam = 0 only the copies are refreshed.
__global__ void k_adam(float* __restrict__ p, const float* __restrict__ gr, float* __restrict__ m1,
                       float* __restrict__ m2, int64_t count, float lr, float c1, float c2, int do_adam, SegTable S) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  float v = p[i];
  if (do_adam) {
    const float gg = gr[i];
    const float a = 0.9f * m1[i] + 0.1f * gg;
    const float b = 0.999f * m2[i] + 0.001f * gg * gg;
    m1[i] = a;
    m2[i] = b;
    v -= lr * (a / c1) / (sqrtf(b / c2) + 1e-8f);
    p[i] = v;
  }
  int l = 0;
  while (l + 1 < S.nl && i >= S.l[l + 1].off) ++l;
  const SegLayer& s = S.l[l];
  int64_t r = i - s.off;
  const int64_t nW1 = (int64_t)s.dA * H, nW2 = (int64_t)H * H, nO = (int64_t)s.dB * NO;
  if (r < nW1) {
    const int a = (int)(r / H), j = (int)(r % H);
    s.W1t[j * KA + a] = (bf16)v;
    s.W1t[j * KA + KLO + a] = (bf16)v;
    s.W1q[((j >> 5) * 64 + a + 16 * ((j >> 3) & 3)) * 8 + (j & 7)] = (bf16)v;
    return;
  }
  r -= nW1 + H;  // b1 is used in FP32 from the master array
  if (r < 0) return;
  if (r < nW2) {
    const int a = (int)(r / H), j = (int)(r % H);
    // wave j >> 6, fragment (j >> 4) & 3, row j & 15
    s.W2p[(((int64_t)(j >> 6) * 8 + (a >> 5)) * 4 + ((j >> 4) & 3)) * 512 + ((j & 15) + 16 * ((a >> 3) & 3)) * 8 +
          (a & 7)] = (bf16)v;
    s.W2q[(((int64_t)(a >> 6) * 8 + (j >> 5)) * 4 + ((a >> 4) & 3)) * 512 + ((a & 15) + 16 * ((j >> 3) & 3)) * 8 +
          (j & 7)] = (bf16)v;
    return;
  }
  r -= nW2 + H;
  if (r < 0) return;
  if (r < H * nO) {
    const int a = (int)(r / nO), o = (int)(r % nO);
    const int c = o / NO, col = o % NO;
    // coordinate c, wave col >> 4, row col & 15; the 65th logit in row c of W3L
    const int kq = c * NOP + col;
    s.W3q[(((int64_t)(kq >> 5) * 4 + (a >> 6)) * 4 + ((a >> 4) & 3)) * 512 + ((a & 15) + 16 * ((kq >> 3) & 3)) * 8 +
          (kq & 7)] = (bf16)v;
    if (col < 64) {
      s.W3p[(((int64_t)c * 4 + (col >> 4)) * 8 + (a >> 5)) * 512 + ((col & 15) + 16 * ((a >> 3) & 3)) * 8 + (a & 7)] =
          (bf16)v;
    } else {
      s.W3L[((a >> 5) * 64 + c + 16 * ((a >> 3) & 3)) * 8 + (a & 7)] = (bf16)v;
    }
    return;
  }
  r -= H * nO;
  s.b3p[(r / NO) * NOP + r % NO] = v;
}

// Initial parameters: the weights of the first two dense layers of every
// coupling layer uniform in +-sqrt(6 / fan_in) from Philox4x64-10 (counter
// (index, 0, 0, 0), key (seed, 3)); biases and the output layer zero, so the
// flow starts as the identity map while every layer's gradient is live.
__global__ void k_init_params(float* __restrict__ p, int64_t count, uint64_t seed, SegTable S) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  int l = 0;
  while (l + 1 < S.nl && i >= S.l[l + 1].off) ++l;
  const SegLayer& s = S.l[l];
  const int64_t r = i - s.off, nW1 = (int64_t)s.dA * H, nW2 = (int64_t)H * H;
  float a = 0.0f;
  if (r < nW1) a = sqrtf(6.0f / (float)s.dA);
  else if (r >= nW1 + H && r < nW1 + H + nW2) a = sqrtf(6.0f / (float)H);
  float v = 0.0f;
  if (a > 0.0f) {
    const U4 q = philox4x64_10((uint64_t)i, 0, 0, 0, seed, 3);
    v = (float)((2.0 * u01(q.x0) - 1.0) * a);
  }
  p[i] = v;
}

}  // namespace flow
}  // namespace mf

using namespace mf;
using namespace mf::flow;

struct mf_flow {
  mf_flow_config cfg;
  int d, nl;
  int64_t count = 0;
  std::vector<std::vector<uint8_t>> mask;
  Layers L;
  SegTable seg;
  int64_t loff[MAXL];
  float* d_p = nullptr;   // masters
  float* d_g = nullptr;   // gradient
  float* d_m1 = nullptr;  // Adam moments
  float* d_m2 = nullptr;
  bf16* d_w16 = nullptr;  // BF16 weight copies of every layer
  float* d_b3p = nullptr;
  int64_t step = 0;
  // training work buffers (max_batch events)
  int64_t cap = 0;
  float* d_lin = nullptr;   // [nl][d][cap] layer inputs
  float* d_y = nullptr;     // [d][cap]
  float* d_gy = nullptr;    // [d][cap]
  float* d_lq = nullptr;    // [cap]
  float* d_weff = nullptr;  // [cap] per-point loss weights of the variance loss
  Operands op{};            // operands of the weight gradients of `group` layers
  int group = 0;
  bf16* d_op = nullptr;
  float* d_part = nullptr;  // partials of the weight gradients, split over events
  size_t part_cap = 0;      // floats
  float* d_scal = nullptr;  // wsum, loss
  std::vector<float*> d_losses;
};

namespace {

// Chunks of events of the weight gradients: at most two workgroups per compute
// unit over the tiles of all layers, so that all run at once (516 workgroups
// for one layer took 69 us, 504 took 57), whole slices per chunk, and at most
// WGRAD_MAX chunks, which the reduction adds up in turn.  A chunk is one FP32
// sum; batches whose chunks would be longer than WGRAD_CHUNK events take
// several such rounds of workgroups instead.
constexpr int64_t WGRAD_BLOCKS = 512;
constexpr int64_t WGRAD_MAX = 64;
constexpr int64_t WGRAD_CHUNK = 16384;

mf_status launch_err(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return set_error(MF_EDEVICE, "%s launch: %s", what, hipGetErrorString(e));
  return MF_OK;
}


// Layers l0 .. l1 - 1, whose operands are held.
WgradArgs wgrad_args(const mf_flow* f, int l0, int l1, int64_t n) {
  WgradArgs a{};
  for (int l = l0; l < l1; ++l) {
    const Operands& o = f->op;
    const bf16* X[3] = {o.h2, o.h1, o.xa};
    const bf16* G[3] = {o.go, o.ga2, o.ga1};
    const int M[3] = {H, H, KA}, N[3] = {f->L.L[l].dB * NOG, H, H};
    for (int k = 0; k < 3; ++k) {
      Product& p = a.p[a.np++];
      p.X = X[k] + (l - l0) * o.stride;
      p.G = G[k] + (l - l0) * o.stride;
      p.M = M[k];
      p.N = N[k];
      p.tiles_n = (p.N + WT - 1) / WT;
      p.first = a.tiles;
      a.tiles += p.tiles_n * ((p.M + WT - 1) / WT);
      p.off = a.zs;
      a.zs += (int64_t)(p.M + 1) * p.N;
    }
  }
  a.n = n;
  const int64_t fit = std::max<int64_t>(1, std::min(WGRAD_BLOCKS / a.tiles, WGRAD_MAX));
  const int64_t rounds = std::min((n + fit * WGRAD_CHUNK - 1) / (fit * WGRAD_CHUNK), WGRAD_MAX / fit);
  const int64_t z = fit * rounds;
  a.zmax = z;
  a.chunk = ((n + z - 1) / z + WK - 1) / WK * WK;
  return a;
}

// Floats of the partials of layers l0 .. l1 - 1 for up to cap events: fewer
// events may take more chunks than cap does, of whole slices.
size_t partials(const mf_flow* f, int l0, int l1, int64_t cap) {
  const WgradArgs a = wgrad_args(f, l0, l1, cap);
  return (size_t)(std::min(a.zmax, (cap + WK - 1) / WK) * a.zs);
}

// Weight and bias gradients of layers l0 .. l1 - 1 over n events from the
// operands.
bool weight_grads(mf_flow* f, int l0, int l1, int64_t n, hipStream_t s) {
  WgradArgs a = wgrad_args(f, l0, l1, n);
  const int64_t Z = (n + a.chunk - 1) / a.chunk;
  // the partials of all chunks must fit the buffer sized at creation
  if ((size_t)(Z * a.zs) > f->part_cap) return false;
  a.part = f->d_part;
  hipLaunchKernelGGL(k_wgrad, dim3((unsigned)(a.tiles * Z)), dim3(256), 0, s, a);
  ReduceArgs r{};
  int64_t most = 0;
  for (int l = l0, k = 0; l < l1; ++l, ++k) {
    r.dA[k] = f->L.L[l].dA;
    r.dB[k] = f->L.L[l].dB;
    r.off[k] = a.p[3 * k].off;
    r.goff[k] = f->loff[l];
    most = std::max(most, (int64_t)(H + 1) * (r.dB[k] * NOG + H) + (int64_t)(r.dA[k] + 1) * H);
  }
  hipLaunchKernelGGL(k_reduce_grad, dim3((unsigned)((most + 255) / 256), (unsigned)(l1 - l0)), dim3(256), 0, s, f->d_part,
                     (int)Z, a.zs, r, f->d_g);
  return true;
}

void run_layers(mf_flow* f, float* y, int64_t n, int64_t ld, float* logq, bool inverse, bool cache, hipStream_t s) {
  const unsigned nblk = (unsigned)((n + T - 1) / T);
  const int64_t ls = (int64_t)f->d * f->cap;
  if (inverse)
    hipLaunchKernelGGL((k_coupling<true, false>), dim3(nblk), dim3(256), 0, s, f->L, f->nl, y, n, ld, logq, f->d_lin, ls,
                       f->d);
  else if (cache)
    hipLaunchKernelGGL((k_coupling<false, true>), dim3(nblk), dim3(256), 0, s, f->L, f->nl, y, n, ld, logq, f->d_lin, ls,
                       f->d);
  else
    hipLaunchKernelGGL((k_coupling<false, false>), dim3(nblk), dim3(256), 0, s, f->L, f->nl, y, n, ld, logq, f->d_lin, ls,
                       f->d);
}

mf_status refresh(mf_flow* f, hipStream_t s, int do_adam, float lr, float c1, float c2) {
  hipLaunchKernelGGL(k_adam, dim3((unsigned)((f->count + 255) / 256)), dim3(256), 0, s, f->d_p, f->d_g, f->d_m1,
                     f->d_m2, f->count, lr, c1, c2, do_adam, f->seg);
  return launch_err("k_adam");
}

mf_status copy_points(mf_flow* f, const float* src, int64_t n, float* dst, hipStream_t s) {
  if (src == dst) return MF_OK;
  hipError_t e = hipMemcpyAsync(dst, src, sizeof(float) * f->d * n, hipMemcpyDeviceToDevice, s);
  if (e != hipSuccess) return set_error(MF_EDEVICE, "copy of points: %s", hipGetErrorString(e));
  return MF_OK;
}

mf_status loss_grad_impl(mf_flow* f, const float* y, int64_t ldy, const float* w_in, int64_t n, int kind,
                         float* loss_dev, hipStream_t s) {
  const int d = f->d;
  hipError_t e = hipMemcpy2DAsync(f->d_y, sizeof(float) * n, y, sizeof(float) * ldy, sizeof(float) * n, d,
                                  hipMemcpyDeviceToDevice, s);
  if (e != hipSuccess) return set_error(MF_EDEVICE, "batch copy: %s", hipGetErrorString(e));
  run_layers(f, f->d_y, n, n, f->d_lq, false, true, s);
  const float* w = w_in;
  if (kind == MF_FLOW_LOSS_VARIANCE) {
    hipLaunchKernelGGL(k_variance_weights, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, w_in, f->d_lq, n,
                       f->d_weff);
    w = f->d_weff;
    hipLaunchKernelGGL(k_relvar, dim3(1), dim3(RB), 0, s, w_in, f->d_weff, n, loss_dev, f->d_scal);
  } else {
    hipLaunchKernelGGL(k_wsum, dim3(1), dim3(RB), 0, s, w, n, f->d_scal);
    hipLaunchKernelGGL(k_loss, dim3(1), dim3(RB), 0, s, w, f->d_lq, n, f->d_scal, loss_dev);
  }
  for (int l1 = f->nl; l1 > 0; l1 -= f->group) {
    const int l0 = std::max(0, l1 - f->group);
    hipLaunchKernelGGL(k_backward, dim3((unsigned)((n + T - 1) / T)), dim3(256), 0, s, f->L, f->nl, l0, l1, f->d_lin,
                       (int64_t)d * f->cap, n, f->d_gy, w, f->d_scal, f->op, d);
    if (!weight_grads(f, l0, l1, n, s))
      return set_error(MF_EINVAL, "weight-gradient partials exceed the flow's buffer");
  }
  return launch_err("flow backward");
}

}  // namespace

namespace mf {
mf_status flow_apply(mf_flow* f, float* y, int64_t n, int64_t ld, float* logq, bool inverse, hipStream_t s) {
  if (n <= 0) return MF_OK;
  run_layers(f, y, n, ld, logq, inverse, false, s);
  return launch_err("k_coupling");
}
mf_status flow_step(mf_flow* f, const float* y, int64_t ld, const float* w, int64_t n, float* loss_dev, double lr,
                    hipStream_t s) {
  if (n < 1 || n > f->cap) return set_error(MF_EINVAL, "batch must be in 1..%lld", (long long)f->cap);
  mf_status st = loss_grad_impl(f, y, ld, w, n, MF_FLOW_LOSS_KL, loss_dev, s);
  if (st != MF_OK) return st;
  return mf_flow_adam_step(f, lr, s);
}
}  // namespace mf

extern "C" {

mf_status mf_flow_create(const mf_flow_config* cfg, mf_flow** out) {
  clear_error();
  if (!cfg || !out) return set_error(MF_EINVAL, "NULL argument");
  *out = nullptr;
  if (cfg->ndim < 2 || cfg->ndim > FMAXD) return set_error(MF_EINVAL, "ndim must be in 2..%d", FMAXD);
  static_assert(FMAXD - 1 <= KLO, "kept coordinates must fit the high half of the first-layer inputs");
  if (cfg->n_layers < 1 || cfg->n_layers > MAXL) return set_error(MF_EINVAL, "n_layers must be in 1..%d", MAXL);
  if (cfg->hidden != H) return set_error(MF_ENOTSUP, "only hidden width %d is built", H);
  if (cfg->bins != KB) return set_error(MF_ENOTSUP, "only %d bins are built", KB);
  if (cfg->max_batch < 1 || cfg->max_batch > (1LL << 24))
    return set_error(MF_EINVAL, "max_batch must be in 1..2^24");
  mf_flow* f = new mf_flow();
  f->cfg = *cfg;
  f->d = cfg->ndim;
  f->nl = cfg->n_layers;
  const int d = f->d;
  int nb = 0;
  while ((1 << nb) < d) ++nb;
  if (nb < 1) nb = 1;
  int64_t off = 0, w16 = 0, b3 = 0, dBmax = 0;
  f->seg.nl = f->nl;
  for (int l = 0; l < f->nl; ++l) {
    std::vector<uint8_t> m(d);
    LayerDev& L = f->L.L[l];
    L.dA = L.dB = 0;
    for (int j = 0; j < d; ++j) {
      const int bit = (j >> (l % nb)) & 1;
      m[j] = (uint8_t)(bit == (((l / nb) % 2 == 0) ? 1 : 0));
      if (m[j]) L.b_idx[L.dB++] = j;
      else L.a_idx[L.dA++] = j;
    }
    f->mask.push_back(m);
    f->loff[l] = off;
    f->seg.l[l].off = off;
    f->seg.l[l].dA = L.dA;
    f->seg.l[l].dB = L.dB;
    off += (int64_t)L.dA * H + H + (int64_t)H * H + H + (int64_t)H * L.dB * NO + L.dB * NO;
    w16 += (int64_t)H * KA + (int64_t)H * H + (int64_t)L.dB * 64 * H + (int64_t)16 * H + (int64_t)H * H +
           (int64_t)(L.dB * NOP + 31) / 32 * 32 * H + (int64_t)16 * H;
    b3 += (int64_t)L.dB * NOP;
    if (L.dB > dBmax) dBmax = L.dB;
  }
  f->count = off;
  auto cleanup = [&](mf_status s) {
    mf_flow_destroy(f);
    return s;
  };
  // the layer kernel keeps the transformed coordinates' inputs in a tile of
  // TBMAX rows (the masks above never transform more than half of 16)
  if (dBmax > TBMAX) return cleanup(set_error(MF_EINVAL, "a layer transforms more than %d coordinates", TBMAX));
  const int64_t cap = cfg->max_batch;
  f->cap = cap;

  // operands of the weight gradients of one layer
  const size_t per_layer = ((size_t)cap * (4 * H + KA + dBmax * NOG) + 127) / 128 * 128;
  if (hipMalloc(&f->d_p, sizeof(float) * off) != hipSuccess || hipMalloc(&f->d_g, sizeof(float) * off) != hipSuccess ||
      hipMalloc(&f->d_m1, sizeof(float) * off) != hipSuccess || hipMalloc(&f->d_m2, sizeof(float) * off) != hipSuccess ||
      hipMalloc(&f->d_w16, sizeof(bf16) * w16) != hipSuccess || hipMalloc(&f->d_b3p, sizeof(float) * b3) != hipSuccess ||
      hipMalloc(&f->d_lin, sizeof(float) * f->nl * d * cap) != hipSuccess ||
      hipMalloc(&f->d_y, sizeof(float) * d * cap) != hipSuccess ||
      hipMalloc(&f->d_gy, sizeof(float) * d * cap) != hipSuccess ||
      hipMalloc(&f->d_lq, sizeof(float) * cap) != hipSuccess ||
      hipMalloc(&f->d_weff, sizeof(float) * cap) != hipSuccess ||
      hipMalloc(&f->d_scal, sizeof(float) * 4) != hipSuccess) {
    hipGetLastError();
    return cleanup(set_error(MF_ENOMEM, "flow allocation failed"));
  }
  // the operands of all layers, so that the backward pass is one launch; of a
  // part of them, in as many launches, where the memory does not hold them
  for (f->group = f->nl;; f->group = (f->group + 1) / 2) {
    f->part_cap = 0;
    for (int l1 = f->nl; l1 > 0; l1 -= f->group)
      f->part_cap = std::max(f->part_cap, partials(f, std::max(0, l1 - f->group), l1, cap));
    const size_t op_bytes = sizeof(bf16) * f->group * per_layer, part_bytes = sizeof(float) * f->part_cap;
    // asked for large flows only: the driver takes a millisecond to say what is free
    size_t avail = SIZE_MAX, total = 0;
    if ((op_bytes < ((size_t)1 << 36) || hipMemGetInfo(&avail, &total) == hipSuccess) &&
        op_bytes + part_bytes <= avail && hipMalloc(&f->d_op, op_bytes) == hipSuccess &&
        hipMalloc(&f->d_part, part_bytes) == hipSuccess)
      break;
    hipGetLastError();
    hipFree(f->d_op);
    f->d_op = nullptr;
    f->d_part = nullptr;
    if (f->group == 1) return cleanup(set_error(MF_ENOMEM, "flow allocation failed"));
  }
  if (hipMemset(f->d_g, 0, sizeof(float) * off) != hipSuccess ||
      hipMemset(f->d_m1, 0, sizeof(float) * off) != hipSuccess ||
      hipMemset(f->d_m2, 0, sizeof(float) * off) != hipSuccess ||
      hipMemset(f->d_w16, 0, sizeof(bf16) * w16) != hipSuccess ||
      hipMemset(f->d_b3p, 0, sizeof(float) * b3) != hipSuccess)
    return cleanup(set_error(MF_EDEVICE, "flow initialisation failed"));
  bf16* wp = f->d_w16;
  float* bp = f->d_b3p;
  f->op.stride = (int64_t)per_layer;
  f->op.h1 = f->d_op;
  f->op.h2 = f->op.h1 + cap * H;
  f->op.ga1 = f->op.h2 + cap * H;
  f->op.ga2 = f->op.ga1 + cap * H;
  f->op.xa = f->op.ga2 + cap * H;
  f->op.go = f->op.xa + cap * KA;
  for (int l = 0; l < f->nl; ++l) {
    LayerDev& L = f->L.L[l];
    L.W1t = wp;
    f->seg.l[l].W1t = wp;
    wp += (int64_t)H * KA;
    L.W2p = wp;
    f->seg.l[l].W2p = wp;
    wp += (int64_t)H * H;
    L.W3p = wp;
    f->seg.l[l].W3p = wp;
    wp += (int64_t)L.dB * 64 * H;
    L.W3L = wp;
    f->seg.l[l].W3L = wp;
    wp += (int64_t)16 * H;
    L.W2q = wp;
    f->seg.l[l].W2q = wp;
    wp += (int64_t)H * H;
    L.W3q = wp;
    f->seg.l[l].W3q = wp;
    wp += (int64_t)(L.dB * NOP + 31) / 32 * 32 * H;
    L.W1q = wp;
    f->seg.l[l].W1q = wp;
    wp += (int64_t)16 * H;
    L.b3p = bp;
    f->seg.l[l].b3p = bp;
    bp += (int64_t)L.dB * NOP;
    L.b1 = f->d_p + f->loff[l] + (int64_t)L.dA * H;
    L.b2 = L.b1 + H + (int64_t)H * H;
  }
  hipLaunchKernelGGL(k_init_params, dim3((unsigned)((off + 255) / 256)), dim3(256), 0, 0, f->d_p, off, cfg->seed,
                     f->seg);
  if (refresh(f, nullptr, 0, 0.0f, 1.0f, 1.0f) != MF_OK || hipDeviceSynchronize() != hipSuccess)
    return cleanup(set_error(MF_EDEVICE, "flow parameter initialisation failed"));
  *out = f;
  return MF_OK;
}

void mf_flow_destroy(mf_flow* f) {
  if (!f) return;
  hipFree(f->d_p);
  hipFree(f->d_g);
  hipFree(f->d_m1);
  hipFree(f->d_m2);
  hipFree(f->d_w16);
  hipFree(f->d_b3p);
  hipFree(f->d_lin);
  hipFree(f->d_y);
  hipFree(f->d_gy);
  hipFree(f->d_lq);
  hipFree(f->d_weff);
  hipFree(f->d_op);
  hipFree(f->d_part);
  hipFree(f->d_scal);
  for (float* p : f->d_losses) hipFree(p);
  delete f;
}

int64_t mf_flow_param_count(const mf_flow* f) { return f ? f->count : -1; }

int mf_flow_ndim(const mf_flow* f) { return f ? f->d : 0; }

mf_status mf_flow_masks(const mf_flow* f, uint8_t* out) {
  clear_error();
  if (!f || !out) return set_error(MF_EINVAL, "NULL argument");
  for (int l = 0; l < f->nl; ++l) std::memcpy(out + (size_t)l * f->d, f->mask[l].data(), f->d);
  return MF_OK;
}

mf_status mf_flow_set_params(mf_flow* f, const float* params, int64_t count) {
  clear_error();
  if (!f || !params) return set_error(MF_EINVAL, "NULL argument");
  if (count != f->count) return set_error(MF_EINVAL, "expected %lld parameters, got %lld", (long long)f->count,
                                          (long long)count);
  if (hipMemcpy(f->d_p, params, sizeof(float) * count, hipMemcpyHostToDevice) != hipSuccess ||
      hipMemset(f->d_m1, 0, sizeof(float) * count) != hipSuccess ||
      hipMemset(f->d_m2, 0, sizeof(float) * count) != hipSuccess)
    return set_error(MF_EDEVICE, "parameter upload failed");
  f->step = 0;
  mf_status st = refresh(f, nullptr, 0, 0.0f, 1.0f, 1.0f);
  if (st != MF_OK) return st;
  if (hipDeviceSynchronize() != hipSuccess) return set_error(MF_EDEVICE, "parameter refresh failed");
  return MF_OK;
}

mf_status mf_flow_get_params(const mf_flow* f, float* params, int64_t count) {
  clear_error();
  if (!f || !params) return set_error(MF_EINVAL, "NULL argument");
  if (count != f->count) return set_error(MF_EINVAL, "expected %lld parameters", (long long)f->count);
  if (hipDeviceSynchronize() != hipSuccess ||
      hipMemcpy(params, f->d_p, sizeof(float) * count, hipMemcpyDeviceToHost) != hipSuccess)
    return set_error(MF_EDEVICE, "parameter download failed");
  return MF_OK;
}

mf_status mf_flow_forward(mf_flow* f, const float* y, int64_t n, float* z, float* logq, void* stream) {
  clear_error();
  if (!f) return set_error(MF_EINVAL, "NULL flow");
  if (n < 0) return set_error(MF_EINVAL, "negative event count");
  if (n == 0) return MF_OK;
  if (!y || !z || !logq) return set_error(MF_EINVAL, "NULL buffer");
  hipStream_t s = (hipStream_t)stream;
  mf_status st = copy_points(f, y, n, z, s);
  if (st != MF_OK) return st;
  run_layers(f, z, n, n, logq, false, false, s);
  return launch_err("k_coupling");
}

mf_status mf_flow_inverse(mf_flow* f, const float* z, int64_t n, float* y, float* logq, void* stream) {
  clear_error();
  if (!f) return set_error(MF_EINVAL, "NULL flow");
  if (n < 0) return set_error(MF_EINVAL, "negative event count");
  if (n == 0) return MF_OK;
  if (!y || !z || !logq) return set_error(MF_EINVAL, "NULL buffer");
  hipStream_t s = (hipStream_t)stream;
  mf_status st = copy_points(f, z, n, y, s);
  if (st != MF_OK) return st;
  run_layers(f, y, n, n, logq, true, false, s);
  return launch_err("k_coupling");
}

mf_status mf_flow_loss_grad(mf_flow* f, const float* y, const float* w, int64_t n, int32_t loss_kind, float* grad,
                            double* loss, void* stream) {
  clear_error();
  if (!f) return set_error(MF_EINVAL, "NULL flow");
  if (n < 1 || n > f->cap) return set_error(MF_EINVAL, "n must be in 1..%lld", (long long)f->cap);
  if (!y || !w) return set_error(MF_EINVAL, "NULL buffer");
  if (loss_kind != MF_FLOW_LOSS_KL && loss_kind != MF_FLOW_LOSS_VARIANCE)
    return set_error(MF_EINVAL, "unknown loss %d", loss_kind);
  hipStream_t s = (hipStream_t)stream;
  mf_status st = loss_grad_impl(f, y, n, w, n, loss_kind, f->d_scal + 1, s);
  if (st != MF_OK) return st;
  if (grad && hipMemcpyAsync(grad, f->d_g, sizeof(float) * f->count, hipMemcpyDeviceToDevice, s) != hipSuccess)
    return set_error(MF_EDEVICE, "gradient copy failed");
  if (loss) {
    float l = 0.0f;
    if (hipMemcpyAsync(&l, f->d_scal + 1, sizeof(float), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
      return set_error(MF_EDEVICE, "loss copy failed");
    *loss = l;
  }
  return MF_OK;
}

mf_status mf_flow_adam_step(mf_flow* f, double lr, void* stream) {
  clear_error();
  if (!f) return set_error(MF_EINVAL, "NULL flow");
  if (!(lr >= 0.0)) return set_error(MF_EINVAL, "learning rate must be >= 0");
  f->step += 1;
  const float c1 = (float)(1.0 - std::pow(0.9, (double)f->step));
  const float c2 = (float)(1.0 - std::pow(0.999, (double)f->step));
  return refresh(f, (hipStream_t)stream, 1, (float)lr, c1, c2);
}

mf_status mf_flow_train(mf_flow* f, const float* y, const float* w, int64_t n, const mf_flow_train_opts* o,
                        double* loss_per_epoch) {
  clear_error();
  if (!f || !o) return set_error(MF_EINVAL, "NULL argument");
  if (!y || !w) return set_error(MF_EINVAL, "NULL buffer");
  if (o->epochs < 1) return set_error(MF_EINVAL, "epochs must be >= 1");
  if (o->batch < 1 || o->batch > f->cap) return set_error(MF_EINVAL, "batch must be in 1..%lld", (long long)f->cap);
  if (n < 1) return set_error(MF_EINVAL, "no training points");
  if (!(o->lr > 0.0) || !(o->lr_final >= 0.0)) return set_error(MF_EINVAL, "invalid learning rates");
  if (o->loss != MF_FLOW_LOSS_KL && o->loss != MF_FLOW_LOSS_VARIANCE)
    return set_error(MF_EINVAL, "unknown loss %d", o->loss);
  hipStream_t s = (hipStream_t)o->stream;
  const int64_t per_epoch = (n + o->batch - 1) / o->batch;
  const int64_t total = per_epoch * o->epochs;
  float* d_loss = nullptr;
  if (hipMalloc(&d_loss, sizeof(float) * total) != hipSuccess) return set_error(MF_ENOMEM, "loss history");
  struct Free {
    float* p;
    ~Free() { (void)hipFree(p); }
  } guard{d_loss};
  int64_t t = 0;
  for (int ep = 0; ep < o->epochs; ++ep) {
    for (int64_t b = 0; b < per_epoch; ++b, ++t) {
      const int64_t off = b * o->batch;
      const int64_t nb = std::min<int64_t>(o->batch, n - off);
      // batch slice of the [d][n] points: rows of nb values with pitch n
      mf_status st = loss_grad_impl(f, y + off, n, w + off, nb, o->loss, d_loss + t, s);
      if (st != MF_OK) return st;
      const double lr = o->lr_final + 0.5 * (o->lr - o->lr_final) * (1.0 + std::cos(M_PI * (double)t / (double)total));
      st = mf_flow_adam_step(f, lr, s);
      if (st != MF_OK) return st;
    }
  }
  std::vector<float> hl((size_t)total);
  if (hipMemcpyAsync(hl.data(), d_loss, sizeof(float) * total, hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    return set_error(MF_EDEVICE, "training failed");
  if (loss_per_epoch)
    for (int ep = 0; ep < o->epochs; ++ep) {
      double a = 0.0;
      for (int64_t b = 0; b < per_epoch; ++b) a += hl[(size_t)(ep * per_epoch + b)];
      loss_per_epoch[ep] = a / (double)per_epoch;
    }
  return MF_OK;
}

}  // extern "C"
