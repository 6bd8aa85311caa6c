// Weight statistics for the unweighting efficiency of a sample: mean,
// maximum, non-zero count (ordered block reductions) and an exact quantile by
// radix selection over order-preserving 64-bit keys of the FP64 weights
// (sign bit flipped for non-negative values, all bits flipped for negative
// ones, so that the unsigned keys sort like the values).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>

#include "../../include/mf.h"
#include "status.h"

namespace {

constexpr int SB = 256;
constexpr int SMAXB = 1024;

// per-block sum and sum of squares (in a fixed order), max, non-zero and
// invalid counts
constexpr int NS = 5;
__global__ void __launch_bounds__(SB) k_wstat_partial(const double* __restrict__ w, int64_t n, double* __restrict__ part) {
  __shared__ double ss[SB], sm[SB], sz[SB], sb[SB], sq[SB];
  const int64_t per = (n + gridDim.x - 1) / gridDim.x;
  const int64_t b0 = (int64_t)blockIdx.x * per, b1 = b0 + per < n ? b0 + per : n;
  double s = 0.0, m = -INFINITY, z = 0.0, bad = 0.0, q = 0.0;
  for (int64_t i = b0 + threadIdx.x; i < b1; i += SB) {
    const double v = w[i];
    if (isnan(v)) {
      bad += 1.0;
      continue;
    }
    s += v;
    q += v * v;
    m = v > m ? v : m;
    z += v != 0.0 ? 1.0 : 0.0;
  }
  ss[threadIdx.x] = s;
  sm[threadIdx.x] = m;
  sz[threadIdx.x] = z;
  sb[threadIdx.x] = bad;
  sq[threadIdx.x] = q;
  __syncthreads();
  for (int st = SB / 2; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) {
      ss[threadIdx.x] += ss[threadIdx.x + st];
      sq[threadIdx.x] += sq[threadIdx.x + st];
      sm[threadIdx.x] = fmax(sm[threadIdx.x], sm[threadIdx.x + st]);
      sz[threadIdx.x] += sz[threadIdx.x + st];
      sb[threadIdx.x] += sb[threadIdx.x + st];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[NS * blockIdx.x + 0] = ss[0];
    part[NS * blockIdx.x + 1] = sm[0];
    part[NS * blockIdx.x + 2] = sz[0];
    part[NS * blockIdx.x + 3] = sb[0];
    part[NS * blockIdx.x + 4] = sq[0];
  }
}

// Totals over the blocks in order, one lane per quantity.  The rows go through
// LDS, so that the chain of additions does not wait for memory: 1024 rows 161
// us with one lane reading them one by one, 24 us now.
__global__ void __launch_bounds__(SB) k_wstat_final(const double* __restrict__ part, int nb, double* __restrict__ out) {
  __shared__ double rows[NS * SMAXB];
  for (int i = threadIdx.x; i < NS * nb; i += SB) rows[i] = part[i];
  __syncthreads();
  const int k = threadIdx.x;
  if (k >= NS) return;
  double a = k == 1 ? -INFINITY : 0.0;
#pragma unroll 8
  for (int b = 0; b < nb; ++b) {
    const double v = rows[NS * b + k];
    a = k == 1 ? fmax(a, v) : a + v;
  }
  out[k] = a;
}

// state: [0] prefix, [1] mask of the fixed high bits, [2] rank still to find,
// then the histogram of the next digit, empty before each k_radix_hist
__global__ void k_radix_init(unsigned long long* state, unsigned long long rank) {
  const int t = threadIdx.x;
  if (t < 3) state[t] = t == 2 ? rank : 0ull;
  state[3 + t] = 0ull;
}

__device__ __forceinline__ unsigned long long order_key(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

__global__ void __launch_bounds__(SB) k_radix_hist(const double* __restrict__ w, int64_t n,
                                                   const unsigned long long* __restrict__ state, int shift,
                                                   unsigned long long* __restrict__ hist) {
  __shared__ unsigned int h[256];
  h[threadIdx.x] = 0u;
  __syncthreads();
  const unsigned long long prefix = state[0], mask = state[1];
  for (int64_t i = (int64_t)blockIdx.x * SB + threadIdx.x; i < n; i += (int64_t)gridDim.x * SB) {
    const unsigned long long key = order_key(w[i]);
    if ((key & mask) == prefix) atomicAdd(&h[(key >> shift) & 255ull], 1u);
  }
  __syncthreads();
  if (h[threadIdx.x]) atomicAdd(&hist[threadIdx.x], (unsigned long long)h[threadIdx.x]);
}

// The digit of the rank: thread t has bucket t, whose range of ranks starts at
// the count of the buckets below it.  Empties the histogram for the next digit.
__global__ void __launch_bounds__(256) k_radix_pick(unsigned long long* __restrict__ hist, unsigned long long* state, int shift) {
  __shared__ unsigned long long tot[4];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const unsigned long long c = hist[t], k = state[2];
  unsigned long long incl = c;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const unsigned long long v = __shfl_up(incl, off);
    incl += lane >= off ? v : 0ull;
  }
  if (lane == 63) tot[wave] = incl;
  hist[t] = 0ull;
  __syncthreads();
  for (int w = 0; w < wave; ++w) incl += tot[w];
  // exactly one bucket holds rank k (k is below the total, the last digit takes the rest)
  if (incl - c <= k && (k < incl || t == 255)) {
    state[0] |= (unsigned long long)t << shift;
    state[1] |= 255ull << shift;
    state[2] = k - (incl - c);
  }
}

// out[k] = sum_e dw[k][e] g[e]: per-block partial sums in a fixed order, then
// one block adds the partials in order.
__global__ void __launch_bounds__(SB) k_vjp_partial(const double* __restrict__ dw, int k, const double* __restrict__ g,
                                                   int64_t n, double* __restrict__ part) {
  __shared__ double sh[SB];
  const int64_t per = (n + gridDim.x - 1) / gridDim.x;
  const int64_t b0 = (int64_t)blockIdx.x * per, b1 = b0 + per < n ? b0 + per : n;
  for (int r = 0; r < k; ++r) {
    double a = 0.0;
    for (int64_t i = b0 + threadIdx.x; i < b1; i += SB) a += dw[(int64_t)r * n + i] * g[i];
    sh[threadIdx.x] = a;
    __syncthreads();
    for (int st = SB / 2; st > 0; st >>= 1) {
      if ((int)threadIdx.x < st) sh[threadIdx.x] += sh[threadIdx.x + st];
      __syncthreads();
    }
    if (threadIdx.x == 0) part[(int64_t)blockIdx.x * k + r] = sh[0];
    __syncthreads();
  }
}
// Totals over the blocks in order, wave r for row r.  The rows' partials go
// through LDS, 1024 at most: 391 rows of 9 took 65 us with one lane per row
// reading them one by one, 8 us now.
__global__ void __launch_bounds__(64) k_vjp_final(const double* __restrict__ part, int nb, int k, double* __restrict__ out) {
  __shared__ double col[SMAXB];
  const int r = blockIdx.x;
  for (int b = threadIdx.x; b < nb; b += 64) col[b] = part[(int64_t)b * k + r];
  __syncthreads();
  if (threadIdx.x != 0) return;
  double a = 0.0;
#pragma unroll 8
  for (int b = 0; b < nb; ++b) a += col[b];
  out[r] = a;
}

}  // namespace

// Blocks of the partial-sum kernels for n events.
static int stat_blocks(int64_t n) { return (int)(n < (int64_t)SMAXB * SB ? (n + SB - 1) / SB : SMAXB); }

extern "C" int64_t mf_vjp_workspace(int32_t k, int64_t n) {
  if (k < 1 || n < 1) return 0;
  return (int64_t)sizeof(double) * stat_blocks(n) * k;
}

extern "C" mf_status mf_vjp(const double* dw, int32_t k, const double* g, int64_t n, double* out, void* work,
                            int64_t work_bytes, void* stream) {
  mf::clear_error();
  if (!dw || !g || !out || !work) return mf::set_error(MF_EINVAL, "NULL argument");
  if (k < 1 || k > 64) return mf::set_error(MF_EINVAL, "k must be in 1..64");
  if (n < 1) return mf::set_error(MF_EINVAL, "n must be >= 1");
  if (work_bytes < mf_vjp_workspace(k, n))
    return mf::set_error(MF_EINVAL, "workspace of %lld bytes, %lld needed", (long long)work_bytes,
                         (long long)mf_vjp_workspace(k, n));
  if (((uintptr_t)work & 7) != 0) return mf::set_error(MF_EINVAL, "workspace not 8-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  const int nb = stat_blocks(n);
  double* part = static_cast<double*>(work);
  hipLaunchKernelGGL(k_vjp_partial, dim3(nb), dim3(SB), 0, s, dw, k, g, n, part);
  hipLaunchKernelGGL(k_vjp_final, dim3(k), dim3(64), 0, s, part, nb, k, out);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return mf::set_error(MF_EDEVICE, "vjp launch: %s", hipGetErrorString(e));
  return MF_OK;
}

extern "C" int64_t mf_weight_stats_workspace(int64_t n) {
  if (n < 1) return 0;
  // partial sums (NS per block and NS for the total), then the radix state
  return (int64_t)sizeof(double) * (NS * stat_blocks(n) + NS) + (int64_t)sizeof(unsigned long long) * (256 + 3);
}

extern "C" mf_status mf_weight_stats(const double* w, int64_t n, double q, double* out, void* work,
                                     int64_t work_bytes, void* stream) {
  mf::clear_error();
  if (!w || !out || !work) return mf::set_error(MF_EINVAL, "NULL argument");
  if (n < 1) return mf::set_error(MF_EINVAL, "n must be >= 1");
  if (!(q > 0.0 && q <= 1.0)) return mf::set_error(MF_EINVAL, "q must be in (0,1]");
  if (work_bytes < mf_weight_stats_workspace(n))
    return mf::set_error(MF_EINVAL, "workspace of %lld bytes, %lld needed", (long long)work_bytes,
                         (long long)mf_weight_stats_workspace(n));
  if (((uintptr_t)work & 7) != 0) return mf::set_error(MF_EINVAL, "workspace not 8-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  const int nb = stat_blocks(n);
  double* part = static_cast<double*>(work);
  unsigned long long* st = reinterpret_cast<unsigned long long*>(part + NS * nb + NS);
  hipLaunchKernelGGL(k_wstat_partial, dim3(nb), dim3(SB), 0, s, w, n, part);
  hipLaunchKernelGGL(k_wstat_final, dim3(1), dim3(SB), 0, s, part, nb, part + NS * nb);
  // rank of the quantile: ceil(q n) - 1
  unsigned long long rank = (unsigned long long)std::ceil(q * (double)n);
  if (rank < 1) rank = 1;
  if (rank > (unsigned long long)n) rank = (unsigned long long)n;
  unsigned long long* hist = st + 3;
  mf_status ret = MF_OK;
  hipLaunchKernelGGL(k_radix_init, dim3(1), dim3(256), 0, s, st, rank - 1);
  for (int shift = 56; shift >= 0; shift -= 8) {
    hipLaunchKernelGGL(k_radix_hist, dim3(nb), dim3(SB), 0, s, w, n, st, shift, hist);
    hipLaunchKernelGGL(k_radix_pick, dim3(1), dim3(256), 0, s, hist, st, shift);
  }
  double tot[NS] = {0, 0, 0, 0, 0};
  unsigned long long res[3] = {0, 0, 0};
  if (hipGetLastError() != hipSuccess ||
      hipMemcpyAsync(tot, part + NS * nb, sizeof(tot), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipMemcpyAsync(res, st, sizeof(res), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    ret = MF_EDEVICE;
  (void)hipStreamSynchronize(s);
  if (ret != MF_OK) return mf::set_error(ret, "weight statistics failed on the device");
  if (tot[3] > 0.0) return mf::set_error(MF_EINVAL, "%.0f weights are NaN", tot[3]);
  out[0] = tot[0] / (double)n;
  out[1] = tot[1];
  double qv;
  const unsigned long long key = res[0];
  unsigned long long bits = (key >> 63) ? (key & 0x7FFFFFFFFFFFFFFFull) : ~key;
  std::memcpy(&qv, &bits, sizeof(qv));
  out[2] = qv;
  out[3] = tot[2];
  const double m1 = tot[0] / (double)n, m2 = tot[4] / (double)n;
  out[4] = m1 != 0.0 ? m2 / (m1 * m1) - 1.0 : 0.0;
  return MF_OK;
}
