// Launcher table: the C ABI reaches the templated kernels of one process
// instance through these function pointers (one translation unit per
// instance keeps compilation parallel).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pipeline.h"

namespace mf {

constexpr int BLOCK = 256;
constexpr int WAVES = BLOCK / 64;
constexpr int MAX_BLOCKS = 2048;
constexpr int PART_HEAD = 8;  // S1 hi, S1 lo, S2 hi, S2 lo, nonzero, nonfinite, pad, pad
constexpr int GV = 10;        // w, dw/dm_t, dw/dtheta_0..7

// ---------------------------------------------------- compensated sums
// Error-free two-sum: a + b = s + e exactly.
__device__ __forceinline__ void two_sum(double a, double b, double& s, double& e) {
  s = a + b;
  double bb = s - a;
  e = (a - (s - bb)) + (b - bb);
}
// Double-double accumulate (hi, lo) += v.
__device__ __forceinline__ void dd_add(double& hi, double& lo, double v) {
  double s, e;
  two_sum(hi, v, s, e);
  lo += e;
  two_sum(s, lo, hi, lo);
}

// Adds one wave's 64 values v (LDS) to the d histograms hist[j][nb] (LDS), lane
// j < d to the bins bins[j stride + k] (LDS, 8-byte aligned) of its dimension,
// in event order: LDS additions without a result, which a wave's LDS
// instructions complete in order, eight bins per read.  The lanes past d add to
// spare[nb], so that there is no divergent region.  As a loop of loads,
// additions and stores every event waited for two LDS latencies, which one
// wave per SIMD does not hide: the iteration kernel of 1e5 g g -> t t~ events
// 28.0 -> 24.5 us, of 1e6 q g -> t t~ q events 727 -> 705 us, and accumulating
// 1e6 staged events 180 -> 96 us.
__device__ __forceinline__ void bin_wave(const unsigned char* bins, int stride, const double* v, double* hist,
                                         double* spare, int d, int nb) {
  typedef __attribute__((address_space(3))) double* P;
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));  // addresses formed here, not kept across the amplitudes
  const bool mine = lane < d;
  const unsigned char* b = bins + (mine ? lane : 0) * stride;
  double* h = mine ? hist + lane * nb : spare + (nb >= 32 ? lane & 31 : 0);
  const unsigned keep = mine ? 255u : 0u;
#pragma unroll 2
  for (int g = 0; g < 64; g += 8) {
    const unsigned lo = *reinterpret_cast<const unsigned*>(b + g), hi = *reinterpret_cast<const unsigned*>(b + g + 4);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const unsigned k = ((i < 4 ? lo : hi) >> (8 * (i & 3))) & keep;
      (void)__builtin_amdgcn_ds_atomic_fadd_f64((P)(h + k), v[g + i]);
    }
  }
}

// Deterministic wave-wide sum of a double with error terms (xor butterfly of
// two-sums); every lane ends with the same (hi, lo).  The butterfly order is
// fixed and two-sum is exact, so the result does not depend on timing.
__device__ __forceinline__ void wave_sum_dd(double v, double& hi, double& lo) {
  double s = v, e = 0.0;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const double so = __shfl_xor(s, off), eo = __shfl_xor(e, off);
    double t, err;
    two_sum(s, so, t, err);
    s = t;
    e = (e + eo) + err;
  }
  hi = s;
  lo = e;
}
// Per-wave double-double accumulator in LDS, updated identically by every
// lane of the wave (all lanes hold the same addend).
__device__ __forceinline__ void lds_dd_accumulate(double* acc, double hi, double lo) {
  double h = acc[0], l = acc[1];
  dd_add(h, l, hi);
  dd_add(h, l, lo);
  acc[0] = h;
  acc[1] = l;
}

// Observable histograms (k_observables): bins per observable and, per
// observable, the lower edge and nbins / (upper - lower edge).
constexpr int N_OBS = 3;
constexpr int MAX_OBS_BINS = 64;
struct ObsSpec {
  int nbins;
  double lo[N_OBS], scale[N_OBS];
};

struct Launchers {
  // false: VEGAS iterations go through the staged path (points kernel ->
  // integrand kernel -> accumulation kernel) instead of the fused kernel
  bool fused;
  // of a fused instance: iterations of up to this many events take the staged
  // path all the same (0: none), where the integrand splits an event over
  // lanes
  int64_t staged_events = 0;
  // selection (k_select_points) then the weights of the kept points
  // (k_integrand); list/cnt/cap as for vegas.  raw (an int, here and in
  // integrand_ws): 1 stores a weight that is not finite as it is, for the
  // accumulation that counts and drops it; 0 stores 0
  void (*integrand)(const DevCfg&, const double*, int64_t, double*, int, int, int*, int*, int64_t, hipStream_t);
  void (*integrand_grad)(const DevCfg&, const double*, int64_t, double*, double*, int, hipStream_t);
  // selection (k_select) then the fused weight kernel (k_vegas) of one
  // iteration; list/cnt/cap: per-block event lists, [nblk][cap] and [nblk]
  void (*vegas)(const DevCfg&, const double*, uint64_t, int64_t, uint64_t, double*, int, int, size_t, int*, int*,
                int64_t, double*, hipStream_t);
  // observable histograms of the kept events of the last fused iteration
  // (their weights from vegas' wk output); per-block partial rows
  void (*observables)(const DevCfg&, const double*, uint64_t, uint64_t, const int*, const int*, int64_t,
                      const double*, const ObsSpec&, double*, int, hipStream_t);
  // selection (k_select) then the derivative estimator over the kept events
  void (*grad_vegas)(const DevCfg&, const double*, uint64_t, int64_t, uint64_t, double*, int, size_t, int*, int*,
                     int64_t, hipStream_t);
  // Multi-kernel integrand with a workspace held by the process handle
  // (*ws, created on first use, released with ws_free); used instead of
  // `integrand` when set.  Synchronises the stream (it reads the number of
  // events that pass the cuts).
  hipError_t (*integrand_ws)(const DevCfg&, const double*, int64_t, double*, int, void**, hipStream_t);
  void (*ws_free)(void*);
};

// One per built instance: g g -> t t~ + ng g in FP64 / FP32 amplitudes, and
// the quark channels in FP64.
Launchers launchers_gg0_f64();
Launchers launchers_gg0_f32();
Launchers launchers_gg1_f64();
Launchers launchers_gg1_f32();
Launchers launchers_gg2_f64();
Launchers launchers_gg2_f32();
Launchers launchers_uu_f64();
Launchers launchers_dd_f64();
// the quark channels with one more light parton (FP64)
Launchers launchers_uug_f64();
Launchers launchers_ddg_f64();
Launchers launchers_qg_f64();
Launchers launchers_gg3_f32();
Launchers launchers_gg3_f64();
// g g -> t t~ g g with the colour sum on the matrix cores (staged kernels)
Launchers launchers_gg2s_f32();
Launchers launchers_gg2s_f64();

}  // namespace mf
