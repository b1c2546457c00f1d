// Chain-quality analysis (paper Sec. 1: the statistical error of a Monte Carlo
// average falls as 1/sqrt(N_indep), N_indep = N_conf / (2 tau_ac); Sec. 2.2 and
// the conclusions: the condensate, zero-momentum two-point functions, the
// autocorrelation time and the effective sample size as analysis quantities).
// All sums in FP64 and in a fixed order, so results are reproducible bit for bit.
#include <algorithm>
#include <cmath>

#include "lfs_common.hpp"

namespace lfs {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr int kAcMaxLag = 8192;  // lags + 1 FP64 quotients in LDS: 64 KB

// Sum over the workgroup: lanes by butterfly, then the waves in index order.
// Every thread of the workgroup must call it; all receive the sum.
__device__ __forceinline__ double block_sum(double v, double* red) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) s += red[w];
  return s;
}

// One workgroup per configuration.  Time slice t (first coordinate t) is the
// contiguous block of `slice` = L^(d-1) sites at t * slice; wave w sums slices
// w, w + 4, ... with its lanes strided over the slice, 16 bytes per lane and
// load when every slice starts 16-byte aligned (vec).  Then M = sum_t Phi(t) / V
// (slices in order) and C(t) = (1/V) sum_t0 Phi(t0) Phi((t0 + t) mod L) by thread t.
template <typename T>
__global__ void __launch_bounds__(kThreads) k_observables(int L, int slice, int vec, const T* __restrict__ phi,
                                                         double* __restrict__ M, double* __restrict__ C) {
  extern __shared__ double Phi[];  // [L]
  constexpr int E = 16 / sizeof(T);  // elements per 16 bytes
  struct alignas(16) Vec { T v[E]; };
  const int b = blockIdx.x, lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  const T* f = phi + (size_t)b * L * slice;
  for (int t = w; t < L; t += kWaves) {
    const T* s = f + (size_t)t * slice;
    double acc = 0.0;
    if (vec) {
      for (int i = lane; i < slice / E; i += kWave) {
        const Vec x = reinterpret_cast<const Vec*>(s)[i];
        double part = 0.0;
#pragma unroll
        for (int e = 0; e < E; ++e) part += (double)x.v[e];
        acc += part;
      }
    } else {
      for (int i = lane; i < slice; i += kWave) acc += (double)s[i];
    }
    acc = wave_sum(acc);
    if (lane == 0) Phi[t] = acc;
  }
  __syncthreads();
  const double V = (double)L * slice;
  if (M && threadIdx.x == 0) {
    double m = 0.0;
    for (int t = 0; t < L; ++t) m += Phi[t];
    M[b] = m / V;
  }
  if (C) {
    for (int t = threadIdx.x; t < L; t += kThreads) {
      double c = 0.0;
      for (int t0 = 0, t1 = t; t0 < L; ++t0, t1 = (t1 + 1 == L ? 0 : t1 + 1)) c += Phi[t0] * Phi[t1];
      C[(size_t)b * L + t] = c / V;
    }
  }
}

// Element k of series s: x[s * ldx + k], or x[s * ldx + index[s * n + k]].
__device__ __forceinline__ int64_t series_at(const int64_t* index, int64_t n, int s, int64_t k) {
  return index ? index[(size_t)s * n + k] : k;
}

// Sum of one of the nsum segments of series s, and whether any of its indices falls
// outside [0, ldx) (kBad) or any of its values is not finite, or so large that a deviation
// might not be (kWild).  Segments rather than one workgroup per series: its gathers are bound
// by latency (65536 elements in one workgroup took 48 us).
constexpr int32_t kBad = 1, kWild = 2;
__global__ void __launch_bounds__(kThreads) k_ac_sums(int64_t n, int64_t per, const double* __restrict__ x,
                                                     int64_t ldx, const int64_t* __restrict__ index,
                                                     double* __restrict__ sums, int32_t* __restrict__ bad) {
  __shared__ double red[kWaves];
  const int s = blockIdx.y, o = blockIdx.y * gridDim.x + blockIdx.x;
  const int64_t k1 = std::min<int64_t>(n, (blockIdx.x + 1) * per);
  double acc = 0.0;
  int32_t f = 0;
#pragma unroll 4
  for (int64_t k = blockIdx.x * per + threadIdx.x; k < k1; k += kThreads) {
    const int64_t j = series_at(index, n, s, k);
    if (j < 0 || j >= ldx) {
      f |= kBad;
    } else {
      const double v = x[(size_t)s * ldx + j];
      f |= fabs(v) <= 1e290 ? 0 : kWild;
      acc += v;
    }
  }
  acc = block_sum(acc, red);
  const bool isbad = __syncthreads_or(f & kBad), wild = __syncthreads_or(f & kWild);
  if (threadIdx.x == 0) {
    sums[o] = acc;
    bad[o] = (isbad ? kBad : 0) | (wild ? kWild : 0);
  }
}

// Mean of a series from its segment sums (at most 64, one per lane, fixed butterfly);
// isbad, wild: any segment is.
__device__ __forceinline__ double series_mean(int64_t n, int nsum, const double* sums, const int32_t* bad, bool& isbad,
                                              bool& wild) {
  const int lane = threadIdx.x & (kWave - 1);
  const int32_t f = lane < nsum ? bad[lane] : 0;
  isbad = __ballot(f & kBad) != 0;
  wild = __ballot(f & kWild) != 0;
  return wave_sum(lane < nsum ? sums[lane] : 0.0) / (double)n;
}

// Lags 0 .. T, at most those of a workgroup, in fours.
__host__ __device__ inline int ac_lags(int T) { return T + 4 < 4 * kThreads ? (T + 4) / 4 * 4 : 4 * kThreads; }

// Partial autocovariance sums of one chunk of elements against i + t, for kThreads groups
// of four consecutive lags: deviations from the mean in LDS, zeros past the series' end.
// A thread slides over the chunk four elements at a time, so its 16 products take four
// 16-byte LDS reads (two of them the same for the whole wave), where a thread per lag took
// two 8-byte reads per product; chunks are short enough to give every CU work: 65536
// elements, 2001 lags, 115 -> 16 us.
__global__ void __launch_bounds__(kThreads) k_ac_partial(int64_t n, int T, int chunk, int nsum,
                                                        const double* __restrict__ x, int64_t ldx,
                                                        const int64_t* __restrict__ index,
                                                        const double* __restrict__ sums,
                                                        const int32_t* __restrict__ bad,
                                                        double* __restrict__ partial) {
  extern __shared__ __align__(16) double d[];  // [2 chunk + lags of the workgroup]
  typedef double f64x2 __attribute__((ext_vector_type(2)));
  const int c = blockIdx.x, s = blockIdx.y, nchunk = gridDim.x, t0 = (blockIdx.z * kThreads + threadIdx.x) * 4;
  const int64_t i0 = (int64_t)c * chunk;
  double* out = partial + ((size_t)s * nchunk + c) * (T + 1);
  bool isbad, wild;
  const double mu = series_mean(n, nsum, sums + (size_t)s * nsum, bad + (size_t)s * nsum, isbad, wild);
  if (isbad) {
    for (int r = 0; r < 4; ++r)
      if (t0 + r <= T) out[t0 + r] = 0.0;
    return;
  }
  // d[q]: element i0 + q for q < chunk, then element i0 + lag0 + q - chunk onwards, where
  // lag0 is the workgroup's first lag
  const int lag0 = blockIdx.z * kThreads * 4, span = chunk + ac_lags(T - lag0);
  for (int q = threadIdx.x; q < chunk + span; q += kThreads) {
    const int64_t k = i0 + (q < chunk ? q : lag0 + q - chunk);
    d[q] = k < n ? x[(size_t)s * ldx + series_at(index, n, s, k)] - mu : 0.0;
  }
  __syncthreads();
  if (wild) {  // the zeros past the end would turn an infinity into a NaN
    for (int t = t0; t < t0 + 4 && t <= T; ++t) {
      const double* b = d + chunk + (t - lag0);
      double acc = 0.0;
      for (int i = 0; i < chunk && i < n - i0 - t; ++i) acc += d[i] * b[i];
      out[t] = acc;
    }
    return;
  }
  if (t0 > T) return;
  const f64x2* a = reinterpret_cast<const f64x2*>(d);
  const f64x2* b = reinterpret_cast<const f64x2*>(d + chunk + 4 * threadIdx.x);
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  f64x2 b0 = b[0], b1 = b[1];
#pragma unroll 2
  for (int i = 0; i < chunk; i += 4) {
    const f64x2 a0 = a[i / 2], a1 = a[i / 2 + 1], b2 = b[i / 2 + 2], b3 = b[i / 2 + 3];
    const double av[4] = {a0[0], a0[1], a1[0], a1[1]};
    const double bv[7] = {b0[0], b0[1], b1[0], b1[1], b2[0], b2[1], b3[0]};
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[r] += av[q] * bv[q + r];
    b0 = b2;
    b1 = b3;
  }
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (t0 + r <= T) out[t0 + r] = acc[r];
}

// Gamma(t) = (chunk partials summed in chunk order within each of four slices, the slices
// in order) / (n - t): 64 lags per workgroup.
__global__ void __launch_bounds__(kThreads) k_ac_gamma(int64_t n, int T, int nchunk, int w_max, int nsum,
                                                      const double* __restrict__ partial,
                                                      const int32_t* __restrict__ bad, double* __restrict__ g,
                                                      double* __restrict__ gamma) {
  __shared__ double sh[kWaves][kWave];
  const int s = blockIdx.y, lane = threadIdx.x & (kWave - 1), sl = threadIdx.x / kWave;
  const int t = blockIdx.x * kWave + lane;
  bool isbad = false;
  for (int k = 0; k < nsum; ++k) isbad |= (bad[(size_t)s * nsum + k] & kBad) != 0;
  double acc = 0.0;
  if (t <= T) {
    const int c1 = (int)((int64_t)nchunk * (sl + 1) / kWaves);
#pragma unroll 8
    for (int c = (int)((int64_t)nchunk * sl / kWaves); c < c1; ++c) acc += partial[((size_t)s * nchunk + c) * (T + 1) + t];
  }
  sh[sl][lane] = acc;
  __syncthreads();
  if (sl != 0) return;
  const double nan = __builtin_nan("");
  double v = sh[0][lane];
#pragma unroll
  for (int k = 1; k < kWaves; ++k) v += sh[k][lane];
  v = isbad ? nan : v / (double)(n - t);
  if (t <= T) g[(size_t)s * (T + 1) + t] = v;
  if (gamma && t <= w_max) gamma[(size_t)s * (w_max + 1) + t] = t <= T ? v : nan;
}

// The Madras-Sokal window by one thread: tau = 1/2 + sum_{t=1}^{W} Gamma(t) / Gamma(0)
// for W = 1, 2, ... until W >= c tau (the quotients formed by all threads).  Series of at
// most kAcFold chunks have no k_ac_gamma launch: their partials are added here, in chunk
// order too, and Gamma kept in gin (64 series of 100: 20 us with that launch, 15 without).
constexpr int kAcFold = 4;
__global__ void __launch_bounds__(kThreads) k_ac_final(int64_t n, int T, int nchunk, int w_max, double cwin, int nsum,
                                                      const double* __restrict__ partial, double* gin,
                                                      const int32_t* __restrict__ bad, double* __restrict__ gamma,
                                                      double* __restrict__ tau,
                                                      int32_t* __restrict__ window, uint8_t* __restrict__ found,
                                                      double* __restrict__ n_indep) {
  extern __shared__ __align__(16) double rho[];  // [T + 1]
  const int s = blockIdx.x;
  double* g = gin + (size_t)s * (T + 1);
  const double nan = __builtin_nan("");
  bool isbad = false;
  for (int k = 0; k < nsum; ++k) isbad |= (bad[(size_t)s * nsum + k] & kBad) != 0;
  if (nchunk <= kAcFold) {
    for (int t = threadIdx.x; t <= T; t += kThreads) {
      double acc = 0.0;
#pragma unroll
      for (int c = 0; c < kAcFold; ++c)
        if (c < nchunk) acc += partial[((size_t)s * nchunk + c) * (T + 1) + t];
      g[t] = isbad ? nan : acc / (double)(n - t);
    }
    __syncthreads();
    if (gamma)
      for (int t = threadIdx.x; t <= w_max; t += kThreads) gamma[(size_t)s * (w_max + 1) + t] = t <= T ? g[t] : nan;
  }
  const double g0 = g[0];
  for (int t = threadIdx.x; t <= T; t += kThreads) rho[t] = g[t] / g0;
  __syncthreads();
  if (threadIdx.x != 0) return;
  double tv = nan, ni = 0.0;
  int W = 0;
  uint8_t fo = 0;
  if (isbad) {
    W = -1;
    ni = nan;
  } else if (g0 != 0.0) {
    tv = 0.5;
    for (W = 1; W <= T; ++W) {
      tv += rho[W];
      if ((double)W >= cwin * tv) {
        fo = 1;
        break;
      }
    }
    if (!fo) W = T;
    ni = (double)n / (2.0 * tv);
  }
  tau[s] = tv;
  if (window) window[s] = W;
  if (found) found[s] = fo;
  if (n_indep) n_indep[s] = ni;
}

// Normalised ESS of series s: (sum e^{w - max})^2 / (n sum e^{2 (w - max)}).  One
// workgroup per series (there is no workspace to combine several in), eight loads of each
// thread in flight: of 256 threads where that is the series, or where the series fill the
// chip (1024 series of 200: 14 us with 1024, 7 with 256; of 3000: 19 and 11), else of 1024
// (65536 log-weights: 72 -> 29 us against 256 threads loading one at a time).
__global__ void __launch_bounds__(1024) k_ess(int64_t n, const double* __restrict__ logw, int64_t ldw,
                                              double* __restrict__ ess) {
  constexpr int U = 8;
  __shared__ double red[16];
  const double* w = logw + (size_t)blockIdx.x * ldw;
  const int64_t step = blockDim.x;
  double mx = -HUGE_VAL;
  for (int64_t k = threadIdx.x; k < n; k += U * step) {
    double v[U];
#pragma unroll
    for (int i = 0; i < U; ++i) v[i] = k + i * step < n ? w[k + i * step] : -HUGE_VAL;
#pragma unroll
    for (int i = 0; i < U; ++i) mx = fmax(mx, v[i]);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, kWave));
  if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = mx;
  __syncthreads();
  mx = red[0];
  for (int i = 1; i < (int)(blockDim.x / kWave); ++i) mx = fmax(mx, red[i]);
  double s1 = 0.0, s2 = 0.0;
  for (int64_t k = threadIdx.x; k < n; k += U * step) {
    double v[U];
#pragma unroll
    for (int i = 0; i < U; ++i) v[i] = k + i * step < n ? w[k + i * step] : -HUGE_VAL;
#pragma unroll
    for (int i = 0; i < U; ++i) {
      if (k + i * step >= n) break;
      const double e = exp(v[i] - mx);
      s1 += e;
      s2 += e * e;
    }
  }
  s1 = lfs::block_sum(s1, red);
  s2 = lfs::block_sum(s2, red);
  if (threadIdx.x == 0) ess[blockIdx.x] = s1 * s1 / ((double)n * s2);
}

struct AcLayout {
  int T, chunk, nchunk, nsum;
  int64_t per;  // elements of a segment sum
  size_t off_bad, off_gamma, off_partial, total;
};

AcLayout ac_layout(int32_t n_series, int64_t n, int32_t w_max) {
  AcLayout a{};
  a.T = (int)std::min<int64_t>(w_max, n - 1);
  // chunks of 512 elements (128 workgroups times the lag groups at 65536), of 2048 in longer
  // series, which fill the chip anyway; a shorter one is cut in four, but not below 128
  const auto up4 = [](int64_t k) { return (int)(k + 3) / 4 * 4; };
  a.chunk = n > 131072 ? 2048 : n > 2048 ? 512 : n > 128 ? std::max(128, up4((n + 3) / 4)) : up4(n);
  a.nchunk = (int)((n + a.chunk - 1) / a.chunk);
  a.nsum = (int)std::min<int64_t>(kWave, (n + 1023) / 1024);
  a.per = (n + a.nsum - 1) / a.nsum;
  const auto up = [](size_t b) { return (b + 255) / 256 * 256; };
  a.off_bad = up((size_t)n_series * a.nsum * sizeof(double));
  a.off_gamma = a.off_bad + up((size_t)n_series * a.nsum * sizeof(int32_t));
  a.off_partial = a.off_gamma + up((size_t)n_series * (a.T + 1) * sizeof(double));
  a.total = a.off_partial + up((size_t)n_series * a.nchunk * (a.T + 1) * sizeof(double));
  return a;
}

bool ac_args_ok(int32_t n_series, int64_t n, int32_t w_max) {
  return n_series >= 1 && n >= 1 && w_max >= 0;
}

}  // namespace
}  // namespace lfs

extern "C" int32_t lfs_observables(int32_t dim, int32_t L, int32_t B, const void* phi, int32_t fp64,
                                   double* M, double* C, void* stream) {
  LFS_RETURN_IF(dim != 2 && dim != 3, LFS_EINVAL);
  LFS_RETURN_IF(L < 2 || B < 0 || !phi || (!M && !C), LFS_EINVAL);
  LFS_RETURN_IF(L > 4096, LFS_EUNSUPPORTED);
  if (B == 0) return LFS_OK;
  const int slice = dim == 2 ? L : L * L;
  const size_t shm = (size_t)L * sizeof(double);
  const int vec = (slice * (fp64 ? 8 : 4)) % 16 == 0 && reinterpret_cast<uintptr_t>(phi) % 16 == 0;
  hipStream_t st = (hipStream_t)stream;
  if (fp64)
    hipLaunchKernelGGL(lfs::k_observables<double>, dim3(B), dim3(lfs::kThreads), shm, st, L, slice, vec,
                       (const double*)phi, M, C);
  else
    hipLaunchKernelGGL(lfs::k_observables<float>, dim3(B), dim3(lfs::kThreads), shm, st, L, slice, vec,
                       (const float*)phi, M, C);
  return lfs::launch_status();
}

extern "C" size_t lfs_autocorr_workspace_bytes(int32_t n_series, int64_t n, int32_t w_max) {
  if (!lfs::ac_args_ok(n_series, n, w_max)) return 0;
  return lfs::ac_layout(n_series, n, w_max).total;
}

extern "C" int32_t lfs_autocorr(int32_t n_series, int64_t n, const double* x, int64_t ldx,
                                const int64_t* index, int32_t w_max, double c, double* gamma,
                                double* tau, int32_t* window, uint8_t* found, double* n_indep,
                                void* ws, size_t ws_bytes, void* stream) {
  LFS_RETURN_IF(!lfs::ac_args_ok(n_series, n, w_max) || !x || !tau || !ws || !(c > 0.0), LFS_EINVAL);
  LFS_RETURN_IF(ldx < 1 || (!index && ldx < n), LFS_EINVAL);
  LFS_RETURN_IF(w_max > lfs::kAcMaxLag || n_series > 65535, LFS_EUNSUPPORTED);
  const lfs::AcLayout a = lfs::ac_layout(n_series, n, w_max);
  LFS_RETURN_IF(ws_bytes < a.total, LFS_EWORKSPACE);
  LFS_RETURN_IF(a.nchunk > (1 << 30), LFS_EUNSUPPORTED);
  char* base = static_cast<char*>(ws);
  double* sums = reinterpret_cast<double*>(base);
  int32_t* bad = reinterpret_cast<int32_t*>(base + a.off_bad);
  double* g = reinterpret_cast<double*>(base + a.off_gamma);
  double* partial = reinterpret_cast<double*>(base + a.off_partial);
  const size_t shm_partial = (size_t)(2 * a.chunk + lfs::ac_lags(a.T)) * sizeof(double);
  const size_t shm_final = (size_t)(a.T + 1) * sizeof(double);
  if (!lfs::set_lds_limit<lfs::k_ac_final>((lfs::kAcMaxLag + 1) * sizeof(double))) return LFS_EDEVICE;
  hipStream_t st = (hipStream_t)stream;
  hipLaunchKernelGGL(lfs::k_ac_sums, dim3(a.nsum, n_series), dim3(lfs::kThreads), 0, st, n, a.per, x, ldx, index, sums,
                     bad);
  hipLaunchKernelGGL(lfs::k_ac_partial, dim3(a.nchunk, n_series, a.T / (4 * lfs::kThreads) + 1), dim3(lfs::kThreads),
                     shm_partial, st, n, a.T, a.chunk, a.nsum, x, ldx, index, sums, bad, partial);
  if (a.nchunk > lfs::kAcFold)
    hipLaunchKernelGGL(lfs::k_ac_gamma, dim3((unsigned)std::max(a.T, gamma ? w_max : 0) / lfs::kWave + 1, n_series),
                       dim3(lfs::kThreads), 0, st, n, a.T, a.nchunk, w_max, a.nsum, partial, bad, g, gamma);
  hipLaunchKernelGGL(lfs::k_ac_final, dim3(n_series), dim3(lfs::kThreads), shm_final, st, n, a.T, a.nchunk, w_max, c,
                     a.nsum, partial, g, bad, gamma, tau, window, found, n_indep);
  return lfs::launch_status();
}

extern "C" int32_t lfs_ess(int32_t n_series, int64_t n, const double* logw, int64_t ldw, double* ess,
                           void* stream) {
  LFS_RETURN_IF(n_series < 1 || n < 1 || ldw < n || !logw || !ess, LFS_EINVAL);
  hipLaunchKernelGGL(lfs::k_ess, dim3(n_series), dim3(n <= 2048 || n_series > 512 ? 256 : 1024), 0,
                     (hipStream_t)stream, n, logw, ldw, ess);
  return lfs::launch_status();
}
