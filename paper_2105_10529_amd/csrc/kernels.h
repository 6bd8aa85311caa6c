// Templated per-event kernels of the integrand library (HIP, gfx950),
// instantiated per process and amplitude precision in the inst_*.hip units
// and reached from the C ABI through the launcher table of launch.h.
#pragma once
#include <hip/hip_runtime.h>

#include "launch.h"
#include "pipeline.h"

namespace mf {
namespace {

// Block-chunked event loops: chunk `it` of this block covers events
// [chunk_base(it), chunk_base(it) + BLOCK).  Both quantities are uniform over
// the block and computed from scalars only.
__device__ __forceinline__ int64_t chunk_base(int64_t it) {
  return (int64_t)blockIdx.x * BLOCK + it * (int64_t)gridDim.x * BLOCK;
}
__device__ __forceinline__ int64_t chunks_of_block(int64_t n) {
  const int64_t b0 = (int64_t)blockIdx.x * BLOCK, stride = (int64_t)gridDim.x * BLOCK;
  return b0 < n ? (n - b0 + stride - 1) / stride : 0;
}

// -------------------------------------------------------------- integrand
// At caller-supplied points: k_select_points writes w = 0 for every point and
// lists, per block and in point order, the points that pass threshold and
// cuts; k_integrand evaluates the weights of the listed points only (full
// wavefronts of points that count, as in the fused iteration).
template <int NG>
__global__ void __launch_bounds__(BLOCK) k_select_points(DevCfg c, const double* __restrict__ u, int64_t n,
                                                         double* __restrict__ w, int* __restrict__ list,
                                                         int* __restrict__ cnt, int64_t cap) {
  __shared__ int wcount[WAVES];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int* out = list + (int64_t)blockIdx.x * cap;
  int qn = 0;
  const int64_t nchunk = chunks_of_block(n);
  for (int64_t it = 0; it < nchunk; ++it) {
    const int64_t e0 = chunk_base(it) + tid;
    const bool live = e0 < n;
    const int64_t e = live ? e0 : n - 1;
    double x[MAXD];
#pragma unroll
    for (int j = 0; j < MAXD; ++j)
      if (j < c.ndim) x[j] = u[(int64_t)j * n + e];
    const bool pass = event_passes<NG>(c, x) && live;
    if (live) w[e0] = 0.0;
    const unsigned long long b = __ballot(pass);
    if (lane == 0) wcount[wave] = __popcll(b);
    __syncthreads();
    int off = qn, total = 0;
#pragma unroll
    for (int v = 0; v < WAVES; ++v) {
      const int cv = wcount[v];
      off += v < wave ? cv : 0;
      total += cv;
    }
    if (pass) out[off + __popcll(b & ((1ull << lane) - 1ull))] = (int)e0;
    __syncthreads();
    qn += total;
  }
  if (tid == 0) cnt[blockIdx.x] = qn;
}

// Running offsets of the selection blocks' lists in LDS: pre[b] is the number
// of entries of the blocks before b, pre[nblk] and what follows the total.  All
// threads of the block take part.
__device__ __forceinline__ void list_offsets(const int* __restrict__ cnt, int nblk, int* pre) {
  constexpr int PER = MAX_BLOCKS / BLOCK;
  __shared__ int wsum[WAVES];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int v[PER], s = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int b = tid * PER + k;
    v[k] = b < nblk ? cnt[b] : 0;
    s += v[k];
  }
  int inc = s;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int o = __shfl_up(inc, off);
    inc += lane >= off ? o : 0;
  }
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  int base = inc - s;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) base += w < wave ? wsum[w] : 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int b = tid * PER + k;
    pre[b] = base;
    base += v[k];
  }
  if (tid == BLOCK - 1) pre[MAX_BLOCKS] = base;
  __syncthreads();
}
// The g-th entry of the lists laid end to end (0 <= g < pre[nblk]).  The search
// takes the same number of steps for every lane, so that the event loops have no
// divergent region.
__device__ __forceinline__ int list_entry(const int* __restrict__ list, int64_t cap, const int* pre, int nblk, int g) {
  // steps 2^k .. 1 with 2^k < nblk: lo + step stays below MAX_BLOCKS, and below
  // nblk where it is taken
  static_assert((MAX_BLOCKS & (MAX_BLOCKS - 1)) == 0, "a power of two");
  int lo = 0;  // the last list with pre[lo] <= g
  for (int step = nblk > 1 ? 1 << (31 - __builtin_clz(nblk - 1)) : 0; step > 0; step >>= 1)
    lo = pre[lo + step] <= g ? lo + step : lo;
  return list[(int64_t)lo * cap + (g - pre[lo])];
}

// Lanes per event of the FP32 g g -> t t~ g g integrand, which deals the 16
// gluon polarisation states out to them: the number that takes the least
// time for nsel events on 1024 SIMDs, one wave each at a time.  Measured, one
// round of the chip takes 25 us for what an event needs once (its
// kinematics, in every lane) and 41 us per state of a lane (16, 4 and 1 lanes
// per event: 70, 195 and 700 us).  65536 points (22900 kept): one lane 714
// us, always four 396, chosen 359; 20000 points 708, 201 and 131 us; 1.5e6
// points stay 1 % faster with four lanes than with one.
__device__ __forceinline__ int state_lanes(int nsel) {
  int best = 4;
  int64_t cost = -1;
  for (int l = 4; l <= 16; l *= 2) {
    const int64_t waves = ((int64_t)nsel * l + 63) / 64, c = (waves + 1023) / 1024 * (25 + 41 * (16 / l));
    if (cost < 0 || c < cost) {
      cost = c;
      best = l;
    }
  }
  return best;
}

// The kept points, numbered through all blocks' lists and dealt out in chunks
// of BLOCK / LANES, so that every block has full chunks whatever share of its
// own points passed (with cuts a chunk of 256 points keeps 90 to 150 of them;
// g g -> t t~ g g FP32 at 2e5 points 2.83 -> 1.47 ms, g g -> t t~ g FP64 at
// 1e6 points 0.56 -> 0.39 ms).  Without final-state partons nearly every point
// passes, and each block takes its own list (g g -> t t~ at 1e6 points 114 us
// against 120 us through the offsets).
template <int NG, int CH, class RA, int LANES>
__device__ __forceinline__ void integrand_loop(const DevCfg& c, const double* __restrict__ u, int64_t n,
                                               double* __restrict__ w, int raw, const int* __restrict__ list,
                                               int64_t cap, const int* pre, int nblk, int nsel) {
  constexpr bool DEALT = NG > 0;
  constexpr int PER = BLOCK / LANES;
  const int* own = list + (int64_t)blockIdx.x * cap;
  const int64_t step = DEALT ? (int64_t)gridDim.x * PER : PER;
  for (int64_t j = DEALT ? (int64_t)blockIdx.x * PER : 0; j < nsel; j += step) {
    const int64_t j0 = j + threadIdx.x / LANES;
    const bool live = j0 < nsel;
    const int g = (int)(live ? j0 : nsel - 1);  // idle lanes recompute the last point
    const int64_t e = DEALT ? list_entry(list, cap, pre, nblk, g) : own[g];
    double x[MAXD];
#pragma unroll
    for (int k = 0; k < MAXD; ++k)
      if (k < c.ndim) x[k] = u[(int64_t)k * n + e];
    EventOut<double> r = event_weight<NG, CH, RA, double, LANES, true>(c, x, c.mt, c.pdfc);
    const double v = raw || isfinite(r.w) ? r.w : 0.0;
    if (live && threadIdx.x % LANES == 0) w[e] = v;
  }
}
// LANES = 0: state_lanes of the number of kept points; raw: a weight that is
// not finite is stored as it is instead of 0.
template <int NG, int CH, class RA, int LANES>
__global__ void __launch_bounds__(BLOCK) k_integrand(DevCfg c, const double* __restrict__ u, int64_t n,
                                                     double* __restrict__ w, int raw,
                                                     const int* __restrict__ list, const int* __restrict__ cnt,
                                                     int nblk, int64_t cap) {
  __shared__ int pre[NG > 0 ? MAX_BLOCKS + 1 : 1];
  if constexpr (NG > 0) list_offsets(cnt, nblk, pre);
  const int nsel = __builtin_amdgcn_readfirstlane(NG > 0 ? pre[nblk] : cnt[blockIdx.x]);
  if constexpr (LANES != 0) {
    integrand_loop<NG, CH, RA, LANES>(c, u, n, w, raw, list, cap, pre, nblk, nsel);
  } else {
    const int lanes = state_lanes(nsel);
    if (lanes == 16) integrand_loop<NG, CH, RA, 16>(c, u, n, w, raw, list, cap, pre, nblk, nsel);
    else if (lanes == 8) integrand_loop<NG, CH, RA, 8>(c, u, n, w, raw, list, cap, pre, nblk, nsel);
    else integrand_loop<NG, CH, RA, 4>(c, u, n, w, raw, list, cap, pre, nblk, nsel);
  }
}

// Derivatives of the event weight: m_t by a dual number through phase space
// and amplitudes, plus the scale derivative of the PDFs when mu = m_t; PDF
// parameters through the collapsed derivative tables.
// KEPT: the point is known to pass the cuts.
template <int NG, int CH, class RA, bool KEPT>
__device__ __forceinline__ void grad_event(const DevCfg& c, const double* x, double& w, double* dw) {
  EventOut<Dual<double>> r = event_weight<NG, CH, RA, Dual<double>, 1, KEPT>(c, x, Dual<double>(c.mt, 1.0), c.pdfc);
  w = r.w.v;
  for (int k = 0; k < 9; ++k) dw[k] = 0.0;
  dw[0] = r.w.d;  // r1, r2 and w are zero for an event that fails, so every term below is 0
  if constexpr (CH == 0) {
    double f1 = hermite_x(c.pdfc, r.t1), f2 = hermite_x(c.pdfc, r.t2);
    if (c.mu_is_mt) dw[0] += r.r1.v * (hermite_x(c.pdfd, r.t1) * f2 + f1 * hermite_x(c.pdfd, r.t2));
    for (int k = 0; k < 5; ++k) {
      const double* T = c.pdft + k * NXK;
      dw[1 + k] = r.r1.v * (hermite_x(T, r.t1) * f2 + f1 * hermite_x(T, r.t2));
    }
  } else if constexpr (CH == 3) {
    // w = r1 (u1 + d1) g2 + r2 g1 (u2 + d2) + r3 2 ub1 g2 + r4 g1 2 ub2
    const double* G = c.pdfc;
    const double *U = c.pdfc + NXK, *D = c.pdfc + 2 * NXK, *A = c.pdfc + 3 * NXK;
    const double g1 = hermite_x(G, r.t1), g2 = hermite_x(G, r.t2);
    const double q1 = hermite_x(U, r.t1) + hermite_x(D, r.t1), q2 = hermite_x(U, r.t2) + hermite_x(D, r.t2);
    const double a1 = 2.0 * hermite_x(A, r.t1), a2 = 2.0 * hermite_x(A, r.t2);
    if (c.mu_is_mt) {
      const double* dG = c.pdfd;
      const double *dU = c.pdfd + NXK, *dD = c.pdfd + 2 * NXK, *dA = c.pdfd + 3 * NXK;
      const double dg1 = hermite_x(dG, r.t1), dg2 = hermite_x(dG, r.t2);
      const double dq1 = hermite_x(dU, r.t1) + hermite_x(dD, r.t1), dq2 = hermite_x(dU, r.t2) + hermite_x(dD, r.t2);
      const double da1 = 2.0 * hermite_x(dA, r.t1), da2 = 2.0 * hermite_x(dA, r.t2);
      dw[0] += r.r1.v * (dq1 * g2 + q1 * dg2) + r.r2.v * (dg1 * q2 + g1 * dq2) + r.r3.v * (da1 * g2 + a1 * dg2) +
               r.r4.v * (dg1 * a2 + g1 * da2);
    }
    for (int k = 0; k < 5; ++k) {
      const double* T = c.pdft + k * NXK;
      const double t1 = hermite_x(T, r.t1), t2 = hermite_x(T, r.t2);
      dw[1 + k] = r.r1.v * q1 * t2 + r.r2.v * t1 * q2 + r.r3.v * a1 * t2 + r.r4.v * t1 * a2;
    }
    const double *TU = c.pdft + 5 * NXK, *TD = c.pdft + 6 * NXK, *TA = c.pdft + 7 * NXK;
    dw[6] = r.r1.v * hermite_x(TU, r.t1) * g2 + r.r2.v * g1 * hermite_x(TU, r.t2);
    dw[7] = r.r1.v * hermite_x(TD, r.t1) * g2 + r.r2.v * g1 * hermite_x(TD, r.t2);
    dw[8] = r.r3.v * 2.0 * hermite_x(TA, r.t1) * g2 + r.r4.v * g1 * 2.0 * hermite_x(TA, r.t2);
  } else {
    const int fq = CH == 1 ? 1 : 2;
    const double* Q = c.pdfc + fq * NXK;
    const double* A = c.pdfc + 3 * NXK;
    double q1 = hermite_x(Q, r.t1), a2 = hermite_x(A, r.t2), a1 = hermite_x(A, r.t1), q2 = hermite_x(Q, r.t2);
    if (c.mu_is_mt) {
      const double* dQ = c.pdfd + fq * NXK;
      const double* dA = c.pdfd + 3 * NXK;
      dw[0] += r.r1.v * (hermite_x(dQ, r.t1) * a2 + q1 * hermite_x(dA, r.t2)) +
               r.r2.v * (hermite_x(dA, r.t1) * q2 + a1 * hermite_x(dQ, r.t2));
    }
    const double* TQ = c.pdft + (CH == 1 ? 5 : 6) * NXK;
    const double* TA = c.pdft + 7 * NXK;
    dw[CH == 1 ? 6 : 7] = r.r1.v * (hermite_x(TQ, r.t1) * a2) + r.r2.v * (a1 * hermite_x(TQ, r.t2));
    dw[8] = r.r1.v * (q1 * hermite_x(TA, r.t2)) + r.r2.v * (hermite_x(TA, r.t1) * q2);
  }
}

// One derivative event per lane; writes its weight and nine derivatives.
template <int NG, int CH, class RA, bool KEPT>
__device__ __forceinline__ void grad_point(const DevCfg& c, const double* __restrict__ u, int64_t n, int64_t e, bool live,
                                           double* __restrict__ w, double* __restrict__ dw) {
  double x[MAXD];
#pragma unroll
  for (int j = 0; j < MAXD; ++j)
    if (j < c.ndim) x[j] = u[(int64_t)j * n + e];
  double ww, d[9];
  grad_event<NG, CH, RA, KEPT>(c, x, ww, d);
  bool ok = isfinite(ww);
  for (int k = 0; k < 9; ++k) ok = ok && isfinite(d[k]);
  if (live) {
    if (w) w[e] = ok ? ww : 0.0;
    for (int k = 0; k < 9; ++k) dw[(int64_t)k * n + e] = ok ? d[k] : 0.0;
  }
}

// Derivatives at given points.  The dual numbers fill the register file (one
// wave per SIMD) and an event costs the same whether it passes the cuts or
// not, so with cuts each block compacts: it tests its share of the points
// (kinematics only), writes zeros for those that fail and queues the others in
// LDS, and evaluates them a full block at a time.  The queue is the block's
// own: the call needs no memory and shares none with others.  GRAD_BLOCKS
// blocks, one per compute unit, with equal contiguous shares: 1e5 points of
// g g -> t t~ g (54 % pass) are one pass of 211 events per block, 366 us
// against 710 us in two rounds of 391 blocks.  Shares have 64 points or more
// and waves without events skip the evaluation: what spills goes through
// memory, and 1000 points take 194 us on 16 waves, 354 us on 1024.  Without
// final-state partons nearly every point passes and the points are taken as
// they come; so are up to a block per compute unit of them with FP32 amplitudes,
// which one round takes either way (g g -> t t~ g at 50000 points that all pass:
// 220 us compacted, 207 as they come; FP64 166 and 149, but at 1000 points 111 and
// 130, and compacted it stays).
constexpr int GRAD_BLOCKS = 256;
template <int NG, int CH, class RA, bool COMPACT>
__global__ void __launch_bounds__(BLOCK) k_integrand_grad(DevCfg c, const double* __restrict__ u, int64_t n,
                                                          double* __restrict__ w, double* __restrict__ dw) {
  if constexpr (!COMPACT) {
    const int64_t nchunk = chunks_of_block(n);
    for (int64_t it = 0; it < nchunk; ++it) {
      const int64_t e0 = chunk_base(it) + threadIdx.x;
      const bool live = e0 < n;
      grad_point<NG, CH, RA, false>(c, u, n, live ? e0 : n - 1, live, w, dw);
    }
  } else {
    __shared__ int queue[2 * BLOCK];  // points that passed, relative to the share
    __shared__ int wcount[WAVES];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t b0 = n * blockIdx.x / gridDim.x, b1 = n * (blockIdx.x + 1) / gridDim.x;
    int have = 0;
    for (int64_t next = b0;;) {
      for (; have < BLOCK && next < b1; next += BLOCK) {
        const int64_t e0 = next + tid;
        const bool live = e0 < b1;
        const int64_t e = live ? e0 : b1 - 1;
        double x[MAXD];
#pragma unroll
        for (int j = 0; j < MAXD; ++j)
          if (j < c.ndim) x[j] = u[(int64_t)j * n + e];
        const bool pass = event_passes<NG>(c, x) && live;
        if (live && !pass) {
          if (w) w[e] = 0.0;
          for (int k = 0; k < 9; ++k) dw[(int64_t)k * n + e] = 0.0;
        }
        const unsigned long long ball = __ballot(pass);
        if (lane == 0) wcount[wave] = __popcll(ball);
        __syncthreads();
        int off = have, total = 0;
#pragma unroll
        for (int v = 0; v < WAVES; ++v) {
          const int cv = wcount[v];
          off += v < wave ? cv : 0;
          total += cv;
        }
        if (pass) queue[off + __popcll(ball & ((1ull << lane) - 1ull))] = (int)(e0 - b0);
        __syncthreads();
        have = __builtin_amdgcn_readfirstlane(have + total);
      }
      if (have == 0) break;
      if (64 * wave < have) {
        const bool live = tid < have;
        grad_point<NG, CH, RA, true>(c, u, n, b0 + queue[live ? tid : 0], live, w, dw);
      }
      // the events of the next pass move to the front
      const int rest = have > BLOCK ? have - BLOCK : 0;
      const int v = queue[BLOCK + (tid < rest ? tid : 0)];
      __syncthreads();
      if (tid < rest) queue[tid] = v;
      __syncthreads();
      have = rest;
    }
  }
}

// ----------------------------------------------------- event selection
// Stage 1 of a VEGAS iteration: every event of the block's chunks (the same
// interleaved chunks as the fused kernel) is drawn, mapped and tested for
// threshold and cuts (kinematics only); the indices of the events that pass
// are written, in event order, to the block's own slice list[b * cap ...]
// and their number to cnt[b].  The fused kernel then evaluates the weight of
// those events only, on full wavefronts; events that fail contribute zero
// to every sum and histogram.
template <int NG>
__global__ void __launch_bounds__(BLOCK) k_select(DevCfg c, const double* __restrict__ edges_g, uint64_t iter,
                                                  int64_t N, uint64_t seed, int* __restrict__ list,
                                                  int* __restrict__ cnt, int64_t cap) {
  extern __shared__ double lds[];
  __shared__ int wcount[WAVES];
  const int d = c.ndim, nb = c.nb;
  double* edges = lds;  // d*(nb+1)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int i = tid; i < d * (nb + 1); i += BLOCK) edges[i] = edges_g[i];
  __syncthreads();
  int* out = list + (int64_t)blockIdx.x * cap;
  int qn = 0;
  const int64_t nchunk = chunks_of_block(N);
  for (int64_t it = 0; it < nchunk; ++it) {
    const int64_t e0 = chunk_base(it) + tid;
    const bool live = e0 < N;
    double y[MAXD], x[MAXD];
    event_uniforms((uint64_t)(live ? e0 : N - 1), iter, seed, 0, d, y);
    double jac = 1.0;
#pragma unroll
    for (int j = 0; j < MAXD; ++j)
      if (j < d) {
        int bin;
        x[j] = vegas_map_dim(edges + j * (nb + 1), nb, y[j], bin, jac);
      }
    const bool pass = event_passes<NG>(c, x) && live;
    const unsigned long long b = __ballot(pass);
    if (lane == 0) wcount[wave] = __popcll(b);
    __syncthreads();
    int off = qn, total = 0;
#pragma unroll
    for (int v = 0; v < WAVES; ++v) {
      const int cv = wcount[v];
      off += v < wave ? cv : 0;
      total += cv;
    }
    if (pass) out[off + __popcll(b & ((1ull << lane) - 1ull))] = (int)e0;
    __syncthreads();
    qn += total;
  }
  if (tid == 0) cnt[blockIdx.x] = qn;
}

// ----------------------------------------------------- fused VEGAS iteration
// Stage 2: the weights of the events k_select kept for this block (chunks of
// BLOCK list entries; the last chunk's idle lanes recompute the block's first
// event with the weight masked).  LISTED = false takes the block's chunks of
// all events as they are, without stage 1: where no final-state partons are cut
// on, 58 to 97 % of the events are above threshold, so that up to two chunks per
// block need as many passes with the selection as without.  5 x 1e5 g g -> t t~
// events 297 us with the selection, 276 us without; 2 x 1e6 events on an
// adapted grid (65 % kept) 344 us with it, 387 us without, on a uniform one 436
// and 393 us.  The observables need the lists.
template <int NG, int CH, class RA, bool LISTED = true>
__global__ void __launch_bounds__(BLOCK) k_vegas(DevCfg c, const double* __restrict__ edges_g, uint64_t iter,
                                                 int64_t N, uint64_t seed, double* __restrict__ partials,
                                                 int pstride, const int* __restrict__ list,
                                                 const int* __restrict__ cnt, int64_t cap,
                                                 double* __restrict__ wk) {
  extern __shared__ double lds[];
  const int d = c.ndim, nb = c.nb;
  double* edges = lds;                             // d*(nb+1)
  double* pdf = edges + d * (nb + 1);              // 4*196
  double* hist = pdf + 4 * NXK;                    // WAVES*d*nb
  double* dummy = hist + WAVES * d * nb;           // WAVES*nb: rows for lanes >= d
  double* wacc = dummy + WAVES * nb;               // WAVES*4 compensated sums
  double* w2s = wacc + WAVES * 4;                  // BLOCK
  double* jac_s = w2s + BLOCK;                     // BLOCK
  double* xs = jac_s + BLOCK;                      // d*BLOCK mapped points
  unsigned char* bins_s = (unsigned char*)(xs + d * BLOCK);  // d*BLOCK
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int i = tid; i < d * (nb + 1); i += BLOCK) edges[i] = edges_g[i];
  for (int i = tid; i < 4 * NXK; i += BLOCK) pdf[i] = c.pdfc[i];
  for (int i = tid; i < WAVES * (d + 1) * nb + WAVES * 4; i += BLOCK) hist[i] = 0.0;
  __syncthreads();
  DevCfg cl = c;
  cl.pdfc = pdf;
  // Nothing per lane is carried from one event chunk to the next: sums go to
  // per-wave LDS accumulators after a deterministic wave reduction, counts are
  // ballots (wave-uniform scalars).
  double* acc = wacc + wave * 4;  // S1 (hi, lo), S2 (hi, lo)
  unsigned long long nnz = 0, nbad = 0;
  double* my_hist = hist + wave * d * nb;
  // The chunk loop is controlled by block-uniform scalars (the length of the
  // block's list), so its counter lives in scalar registers and is not
  // exposed to vector-register spills inside the divergent per-event code.
  const int* mine_list = list + (int64_t)blockIdx.x * cap;
  const int nsel = LISTED ? __builtin_amdgcn_readfirstlane(cnt[blockIdx.x]) : 0;
  const int64_t nchunk = LISTED ? (nsel + BLOCK - 1) / BLOCK : chunks_of_block(N);
  for (int64_t it = 0; it < nchunk; ++it) {
    const int64_t j0 = (LISTED ? it * BLOCK : chunk_base(it)) + tid;
    const bool live = j0 < (LISTED ? (int64_t)nsel : N);
    const int64_t e = LISTED ? (int64_t)mine_list[live ? j0 : 0] : (live ? j0 : N - 1);
    {
      // map the uniforms and stage the bin indices and the Jacobian in LDS
      // before the amplitude, so no per-lane value is live across it
      int bins[MAXD];
      double y[MAXD];
      event_uniforms((uint64_t)e, iter, seed, 0, d, y);
      double jac = 1.0;
#pragma unroll
      for (int j = 0; j < MAXD; ++j)
        if (j < d) xs[j * BLOCK + tid] = vegas_map_dim(edges + j * (nb + 1), nb, y[j], bins[j], jac);
#pragma unroll
      for (int j = 0; j < MAXD; ++j)
        if (j < d) bins_s[j * BLOCK + tid] = (unsigned char)bins[j];
      jac_s[tid] = jac;
    }
    asm volatile("" ::: "memory");
    double x[MAXD];
#pragma unroll
    for (int j = 0; j < MAXD; ++j)
      if (j < d) x[j] = xs[j * BLOCK + tid];
    EventOut<double> r = event_weight<NG, CH, RA, double, 1, LISTED>(cl, x, c.mt, pdf);
    asm volatile("" ::: "memory");
    double w = r.w * jac_s[tid];
    const bool finite = isfinite(w);
    nbad += __popcll(__ballot(live && !finite));
    w = (live && finite) ? w : 0.0;
    nnz += __popcll(__ballot(w != 0.0));
    if (LISTED && wk != nullptr && live) wk[(int64_t)blockIdx.x * cap + j0] = w;  // for the observable histograms
    {
      double h1, l1, h2, l2;
      wave_sum_dd(w, h1, l1);
      wave_sum_dd(w * w, h2, l2);
      lds_dd_accumulate(acc, h1, l1);
      lds_dd_accumulate(acc + 2, h2, l2);
    }
    // stage this wave's 64 weights, then bin them in event order
    w2s[tid] = w * w;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    bin_wave(bins_s + wave * 64, BLOCK, w2s + wave * 64, my_hist, dummy + wave * nb, d, nb);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  __syncthreads();
  // combine the wave histograms in wave order, then the compensated sums in
  // thread order (a fixed order: the partials are bitwise reproducible)
  double* p = partials + (int64_t)blockIdx.x * pstride;
  for (int i = tid; i < d * nb; i += BLOCK) {
    double h = 0.0;
    for (int v = 0; v < WAVES; ++v) h += hist[v * d * nb + i];
    p[PART_HEAD + i] = h;
  }
  __syncthreads();
  // counts: wave-uniform per wave; combine the four waves in order
  unsigned long long* ci = (unsigned long long*)w2s;
  if (lane == 0) {
    ci[wave] = nnz;
    ci[WAVES + wave] = nbad;
  }
  __syncthreads();
  if (tid == 0) {
    double acc_hi[2] = {0.0, 0.0}, acc_lo[2] = {0.0, 0.0};
    unsigned long long tn = 0, tb = 0;
    for (int v = 0; v < WAVES; ++v) {
      dd_add(acc_hi[0], acc_lo[0], wacc[4 * v + 0]);
      dd_add(acc_hi[0], acc_lo[0], wacc[4 * v + 1]);
      dd_add(acc_hi[1], acc_lo[1], wacc[4 * v + 2]);
      dd_add(acc_hi[1], acc_lo[1], wacc[4 * v + 3]);
      tn += ci[v];
      tb += ci[WAVES + v];
    }
    p[0] = acc_hi[0];
    p[1] = acc_lo[0];
    p[2] = acc_hi[1];
    p[3] = acc_lo[1];
    p[4] = (double)tn;
    p[5] = (double)tb;
  }
}

// ------------------------------------------------- observable histograms
// Weighted histograms of three observables of the kept events of one fused
// iteration (after k_vegas wrote their weights wk, in list order): 0 = top
// transverse momentum, 1 = invariant mass of the top pair, 2 = transverse
// momentum of the hardest gluon (absent without final gluons).  All three
// are invariant under the longitudinal boost, so they are taken from the
// partonic centre-of-mass momenta of the phase-space map.  Per bin the sum
// of w and of w^2; bin k = floor((v - lo) scale), kept for 0 <= k < nbins.
// One wave's 64 events are staged in LDS and binned by lanes 0..2 (one
// observable each) in event order, so the block partials are reproducible.
template <int NG>
__global__ void __launch_bounds__(BLOCK) k_observables(DevCfg c, const double* __restrict__ edges_g, uint64_t iter,
                                                       uint64_t seed, const int* __restrict__ list,
                                                       const int* __restrict__ cnt, int64_t cap,
                                                       const double* __restrict__ wk, ObsSpec o,
                                                       double* __restrict__ opart) {
  extern __shared__ double lds[];
  const int d = c.ndim, nb = c.nb, onb = o.nbins;
  const int W = N_OBS * onb * 2;
  double* edges = lds;                       // d*(nb+1)
  double* hw = edges + d * (nb + 1);         // [WAVES][N_OBS][onb][2]
  double* ws = hw + WAVES * W;               // [BLOCK] staged weights
  int* ks = (int*)(ws + BLOCK);              // [N_OBS][BLOCK] staged bins
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int i = tid; i < d * (nb + 1); i += BLOCK) edges[i] = edges_g[i];
  for (int i = tid; i < WAVES * W; i += BLOCK) hw[i] = 0.0;
  __syncthreads();
  const int* mine_list = list + (int64_t)blockIdx.x * cap;
  const double* mine_w = wk + (int64_t)blockIdx.x * cap;
  const int nsel = __builtin_amdgcn_readfirstlane(cnt[blockIdx.x]);
  const int64_t nchunk = (nsel + BLOCK - 1) / BLOCK;
  for (int64_t it = 0; it < nchunk; ++it) {
    const int64_t j0 = it * BLOCK + tid;
    const bool live = j0 < nsel;
    const int64_t e = mine_list[live ? j0 : 0];
    double y[MAXD], x[MAXD];
    event_uniforms((uint64_t)e, iter, seed, 0, d, y);
    double jac = 1.0;
#pragma unroll
    for (int j = 0; j < MAXD; ++j)
      if (j < d) {
        int bin;
        x[j] = vegas_map_dim(edges + j * (nb + 1), nb, y[j], bin, jac);
      }
    const double thr = 4.0 * c.mt * c.mt, shat = x[0] * x[1] * c.s;
    V4<double> gl[NG > 0 ? NG : 1], top, atop;
    (void)phase_space<double>(NG, x, shat > thr ? shat : thr * (1.0 + 1e-3), c.mt, gl, top, atop);
    double v[N_OBS];
    v[0] = sqrt(top.x * top.x + top.y * top.y);
    const V4<double> P = top + atop;
    v[1] = sqrt(fmax(mdot(P, P), 0.0));
    v[2] = -1.0;
#pragma unroll
    for (int i = 0; i < NG; ++i) v[2] = fmax(v[2], sqrt(gl[i].x * gl[i].x + gl[i].y * gl[i].y));
    ws[tid] = live ? mine_w[j0] : 0.0;
#pragma unroll
    for (int q = 0; q < N_OBS; ++q) {
      const double t = (v[q] - o.lo[q]) * o.scale[q];
      ks[q * BLOCK + tid] = (live && t >= 0.0 && t < (double)onb) ? (int)t : -1;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (lane < N_OBS) {
      double* h = hw + wave * W + lane * onb * 2;
      const int* kq = ks + lane * BLOCK + wave * 64;
      const double* wq = ws + wave * 64;
      for (int k = 0; k < 64; ++k) {
        const int b = kq[k];
        if (b >= 0) {
          h[2 * b] += wq[k];
          h[2 * b + 1] += wq[k] * wq[k];
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  __syncthreads();
  for (int i = tid; i < W; i += BLOCK) {
    double h = 0.0;
    for (int v2 = 0; v2 < WAVES; ++v2) h += hw[v2 * W + i];
    opart[(int64_t)blockIdx.x * W + i] = h;
  }
}

// ------------------------------------------------- gradient estimator
template <int NG, int CH, class RA>
__global__ void __launch_bounds__(BLOCK) k_grad_vegas(DevCfg c, const double* __restrict__ edges_g, uint64_t iter,
                                                      int64_t N, uint64_t seed, double* __restrict__ partials,
                                                      const int* __restrict__ list, const int* __restrict__ cnt,
                                                      int64_t cap) {
  extern __shared__ double lds[];
  const int d = c.ndim, nb = c.nb;
  const int tid = threadIdx.x, wave = tid >> 6;
  double* edges = lds;
  double* wacc = lds + d * (nb + 1);  // [WAVES][GV][4]: sum (hi, lo), sum of squares (hi, lo)
  for (int i = tid; i < d * (nb + 1); i += BLOCK) edges[i] = edges_g[i];
  for (int i = tid; i < WAVES * GV * 4; i += BLOCK) wacc[i] = 0.0;
  __syncthreads();
  double* acc = wacc + wave * GV * 4;
  // As in k_vegas, nothing per lane is carried across event chunks.
  // Only the events k_select kept: the others have zero weight and zero
  // pathwise derivatives (the cut boundaries do not move with the grid and
  // uniforms frozen).
  const int* mine_list = list + (int64_t)blockIdx.x * cap;
  const int nsel = __builtin_amdgcn_readfirstlane(cnt[blockIdx.x]);
  const int64_t nchunk = (nsel + BLOCK - 1) / BLOCK;
  for (int64_t it = 0; it < nchunk; ++it) {
    const int64_t j0 = it * BLOCK + tid;
    const bool live = j0 < nsel;
    const int64_t e = mine_list[live ? j0 : 0];
    double y[MAXD], x[MAXD];
    int bins[MAXD];
    event_uniforms((uint64_t)e, iter, seed, 0, d, y);
    double jac = 1.0;
#pragma unroll
    for (int j = 0; j < MAXD; ++j)
      if (j < d) x[j] = vegas_map_dim(edges + j * (nb + 1), nb, y[j], bins[j], jac);
    double v[GV];
    grad_event<NG, CH, RA, false>(c, x, v[0], v + 1);
    bool ok = live;
    for (int k = 0; k < GV; ++k) ok = ok && isfinite(v[k]);
    for (int k = 0; k < GV; ++k) {
      const double t = ok ? v[k] * jac : 0.0;
      double h, l;
      wave_sum_dd(t, h, l);
      lds_dd_accumulate(acc + 4 * k, h, l);
      wave_sum_dd(t * t, h, l);
      lds_dd_accumulate(acc + 4 * k + 2, h, l);
    }
  }
  __syncthreads();
  if (tid < GV) {
    const int k = tid;
    double hs = 0.0, ls = 0.0, hq = 0.0, lq = 0.0;
    for (int v = 0; v < WAVES; ++v) {
      const double* a = wacc + v * GV * 4 + 4 * k;
      dd_add(hs, ls, a[0]);
      dd_add(hs, ls, a[1]);
      dd_add(hq, lq, a[2]);
      dd_add(hq, lq, a[3]);
    }
    double* p = partials + (int64_t)blockIdx.x * (3 * GV);
    p[3 * k] = hs;
    p[3 * k + 1] = ls;
    p[3 * k + 2] = hq + lq;
  }
}

}  // namespace

// Launcher table of one (final gluons, channel, amplitude type) instance;
// GRAD = 0 leaves the derivative kernels out, FUSED = 0 the fused iteration;
// LANES: lanes per event of the integrand at given points (0: state_lanes).
template <int NG, int CH, class RA, class RD, int GRAD, int FUSED = 1, int LANES = 1>
Launchers make_launchers() {
  Launchers L;
  L.fused = FUSED != 0;
  // one lane per event leaves part of the chip's 65536 lanes idle (FP32
  // g g -> t t~ g g, two iterations of 2000 events 1.66 -> 0.43 ms, of 1e5
  // events 3.16 -> 2.29 ms; from 1.4e5 events the fused kernel is as fast)
  L.staged_events = LANES == 0 ? 1 << 17 : 0;
  L.integrand = [](const DevCfg& c, const double* u, int64_t n, double* w, int raw, int nblk, int* list, int* cnt,
                   int64_t cap, hipStream_t s) {
    hipLaunchKernelGGL((k_select_points<NG>), dim3(nblk), dim3(BLOCK), 0, s, c, u, n, w, list, cnt, cap);
    // enough blocks for every kept point, four per compute unit at most (the
    // kernels hold one to three; more would only repeat the offsets)
    const int64_t want = (n * (LANES ? LANES : 16) + BLOCK - 1) / BLOCK;
    const unsigned grid = NG == 0 ? (unsigned)nblk : (unsigned)(want < 1024 ? want : 1024);
    hipLaunchKernelGGL((k_integrand<NG, CH, RA, LANES>), dim3(grid), dim3(BLOCK), 0, s, c, u, n, w, raw, list, cnt,
                       nblk, cap);
  };
  L.vegas = nullptr;
  if constexpr (FUSED != 0) {
    L.vegas = [](const DevCfg& c, const double* edges, uint64_t iter, int64_t N, uint64_t seed, double* part,
                 int pstride, int nblk, size_t lds, int* list, int* cnt, int64_t cap, double* wk, hipStream_t s) {
      if constexpr (NG == 0) {
        if (wk == nullptr && N <= 2 * (int64_t)nblk * BLOCK) {
          hipLaunchKernelGGL((k_vegas<NG, CH, RA, false>), dim3(nblk), dim3(BLOCK), lds, s, c, edges, iter, N, seed, part,
                             pstride, list, cnt, cap, wk);
          return;
        }
      }
      hipLaunchKernelGGL((k_select<NG>), dim3(nblk), dim3(BLOCK), sizeof(double) * c.ndim * (c.nb + 1), s, c, edges,
                         iter, N, seed, list, cnt, cap);
      hipLaunchKernelGGL((k_vegas<NG, CH, RA>), dim3(nblk), dim3(BLOCK), lds, s, c, edges, iter, N, seed, part, pstride,
                         list, cnt, cap, wk);
    };
  }
  L.observables = [](const DevCfg& c, const double* edges, uint64_t iter, uint64_t seed, const int* list,
                     const int* cnt, int64_t cap, const double* wk, const ObsSpec& o, double* opart, int nblk,
                     hipStream_t s) {
    const size_t lds = sizeof(double) * ((size_t)c.ndim * (c.nb + 1) + (size_t)WAVES * N_OBS * o.nbins * 2 + BLOCK) +
                       sizeof(int) * N_OBS * BLOCK;
    hipLaunchKernelGGL((k_observables<NG>), dim3(nblk), dim3(BLOCK), lds, s, c, edges, iter, seed, list, cnt, cap, wk,
                       o, opart);
  };
  L.integrand_grad = nullptr;
  L.grad_vegas = nullptr;
  L.integrand_ws = nullptr;
  L.ws_free = nullptr;
  if constexpr (GRAD != 0) {
    L.integrand_grad = [](const DevCfg& c, const double* u, int64_t n, double* w, double* dw, int nblk,
                          hipStream_t s) {
      constexpr bool PLAIN = NG == 0 || std::is_same<RD, Dual<float>>::value;
      if constexpr (PLAIN) {
        if (NG == 0 || n <= (int64_t)GRAD_BLOCKS * BLOCK) {
          hipLaunchKernelGGL((k_integrand_grad<NG, CH, RD, false>), dim3(nblk), dim3(BLOCK), 0, s, c, u, n, w, dw);
          return;
        }
      }
      if constexpr (NG > 0) {
        const unsigned grid = (unsigned)((n + 63) / 64 < GRAD_BLOCKS ? (n + 63) / 64 : GRAD_BLOCKS);
        hipLaunchKernelGGL((k_integrand_grad<NG, CH, RD, true>), dim3(grid), dim3(BLOCK), 0, s, c, u, n, w, dw);
      }
    };
    L.grad_vegas = [](const DevCfg& c, const double* edges, uint64_t iter, int64_t N, uint64_t seed, double* part,
                      int nblk, size_t lds, int* list, int* cnt, int64_t cap, hipStream_t s) {
      hipLaunchKernelGGL((k_select<NG>), dim3(nblk), dim3(BLOCK), sizeof(double) * c.ndim * (c.nb + 1), s, c, edges,
                         iter, N, seed, list, cnt, cap);
      hipLaunchKernelGGL((k_grad_vegas<NG, CH, RD>), dim3(nblk), dim3(BLOCK), lds, s, c, edges, iter, N, seed, part,
                         list, cnt, cap);
    };
  }
  return L;
}

}  // namespace mf
