// Finite-size-scaling analysis of per-sweep (E, M) series.
//
// The paper locates T_C where the Binder cumulants U4 = 1 - <M^4>/(3<M^2>^2)
// (section 2, Eq. (2)) of different lattice sizes cross.  Turning the
// batched simulations' series into those curves takes three steps:
//
//  * k_reweight (device, fp64): single-histogram reweighting (Ferrenberg and
//    Swendsen, PRL 61, 2635 (1988)) of each series sampled at beta0 to a
//    target beta, accumulated as five sums per block of consecutive kept
//    sweeps.  The series stay where the sweeps wrote them.
//  * ising_fss_moments (host): U4, <E>/N and <|M|>/N from the totals and
//    their delete-one-block jackknife errors (B sets of a few numbers).
//  * ising_binder_crossing (host): where two U4 curves on a common grid
//    cross, with the jackknife error from the replica curves.
//
// Definitions (the same in the test oracle, written separately):
//   kept sweeps t = discard .. n-1, count = n - discard; sample j = t -
//   discard is in block floor(j B / count);
//   x_t = -(beta - beta0)(E_t - E_ref), E_ref = E of the first kept sweep;
//   w_t = exp(x_t - max x); sums per block: w, w|M|, w M^2, w M^4, w E with
//   m = double(M), m2 = m m, m4 = m2 m2.
#include <hip/hip_runtime.h>

#include <cmath>
#include <complex>
#include <cstring>
#include <limits>
#include <vector>

#include "ising.h"
#include "ising_runtime.hpp"

namespace ising {
namespace {

constexpr int kRwThreads = 256;
constexpr int kRwMaxBlocks = 4096;
// Blocks of a call up to which each has a workgroup of its own (k_reweight):
// sixteen per compute unit.
constexpr int64_t kRwFewBlocks = 4096;

struct RwLattice {
  const int64_t* EM;  // n x (E, M)
  int64_t n;
  int64_t discard;
  double beta0;
  int64_t used;          // some task reweights it
  int64_t E_min, E_max;  // over the kept sweeps (written by k_series_range where used)
};
struct RwTask {
  int32_t lattice;
  int32_t pad;
  double beta;
};

__device__ __forceinline__ double wave_add(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// One workgroup per series: the least and the greatest E of its kept sweeps
// (a series that no task uses is not read).
__global__ __launch_bounds__(kRwThreads) void k_series_range(RwLattice* lat) {
  __shared__ int64_t red[2][kRwThreads / 64];
  RwLattice* lt = &lat[blockIdx.x];
  if (!lt->used) return;
  const int64_t* EM = lt->EM;
  int64_t lo = std::numeric_limits<int64_t>::max(), hi = std::numeric_limits<int64_t>::min();
  for (int64_t t = lt->discard + threadIdx.x; t < lt->n; t += kRwThreads) {
    const int64_t E = EM[2 * t];
    lo = E < lo ? E : lo;
    hi = E > hi ? E : hi;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const int64_t a = __shfl_xor(lo, off, 64), b = __shfl_xor(hi, off, 64);
    lo = a < lo ? a : lo;
    hi = b > hi ? b : hi;
  }
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = lo;
    red[1][threadIdx.x >> 6] = hi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < kRwThreads / 64; ++i) {
      lo = red[0][i] < lo ? red[0][i] : lo;
      hi = red[1][i] > hi ? red[1][i] : hi;
    }
    lt->E_min = lo;
    lt->E_max = hi;
  }
}

// The five sums of every block of sweeps of a task (lattice, target beta).
// The maximum exponent needs no pass of its own: -db (E - E_ref) is monotone
// in E (E is exact in binary64, and rounding a product is monotone), so it is
// the exponent of E_min or E_max.
//
// Many blocks in all (SHARED false): a workgroup per task, a wave per block.
// A wave reduces its own block, so there is no block barrier, and the
// shuffles are paid once per block of sweeps (a workgroup per block of 400
// sweeps paid them in each of its four waves, after two steps of 256 lanes of
// which the second was nearly half idle).  1743 tasks of 8000 sweeps in 20
// blocks: 148 us -> 51 us, plus 16 us for the series' ranges.
//
// Few blocks (SHARED): a workgroup per task and block, whose waves share it.
// A wave per block would leave most of the chip, and with fewer than four
// blocks per task waves of its own workgroup, without work.  Calls of 10^6
// sweeps with a wave and a workgroup per block: 1 task, 1 block 6.3 -> 2.4 ms
// (half of it the range); 8 tasks, 5 blocks 3.3 -> 1.3; 64 tasks of 10^5
// sweeps, 1 block 0.40 -> 0.18.  At the limit both take the same: 200 and 210
// tasks of 8000 sweeps in 20 blocks 70 and 72 us either way.
template <bool SHARED>
__global__ __launch_bounds__(kRwThreads) void k_reweight(const RwLattice* lat, const RwTask* task,
                                                         int nblocks, double* sums,
                                                         double* shift) {
  // every product and sum rounds on its own, as in the definition above (a
  // fused multiply-add would move the exponent by an ulp of |x|, which is
  // then amplified by exp)
#pragma clang fp contract(off)
  constexpr int kWaves = kRwThreads / 64;
  __shared__ double red[SHARED ? kWaves : 1][5];
  const RwTask tk = task[blockIdx.x];
  const RwLattice lt = lat[tk.lattice];
  const int64_t* EM = lt.EM;
  const int64_t t0 = lt.discard;
  const int64_t count = lt.n - t0;
  const int64_t E_ref = EM[2 * t0];
  const double db = tk.beta - lt.beta0;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const double xm = fmax(-db * (double)(lt.E_min - E_ref), -db * (double)(lt.E_max - E_ref));

  for (int b = SHARED ? (int)blockIdx.y : wave; b < nblocks; b += SHARED ? nblocks : kWaves) {
    const int64_t j0 = ((int64_t)b * count + nblocks - 1) / nblocks;
    const int64_t j1 = ((int64_t)(b + 1) * count + nblocks - 1) / nblocks;
    double s[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (int64_t j = j0 + (SHARED ? (int)threadIdx.x : lane); j < j1;
         j += SHARED ? kRwThreads : 64) {
      const int64_t E = EM[2 * (t0 + j)];
      const double m = (double)EM[2 * (t0 + j) + 1];
      const double x = -db * (double)(E - E_ref);
      const double w = exp(x - xm);
      const double m2 = m * m;
      s[0] += w;
      s[1] += w * fabs(m);
      s[2] += w * m2;
      s[3] += w * (m2 * m2);
      s[4] += w * (double)E;
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) s[i] = wave_add(s[i]);
    double* out = sums + ((int64_t)blockIdx.x * nblocks + b) * 5;
    if (SHARED) {
      if (lane == 0)
        for (int i = 0; i < 5; ++i) red[wave][i] = s[i];
      __syncthreads();
      if (threadIdx.x < 5) {
        double v = 0.0;
        for (int k = 0; k < kWaves; ++k) v += red[k][threadIdx.x];
        out[threadIdx.x] = v;
      }
    } else if (lane == 0) {
      for (int i = 0; i < 5; ++i) out[i] = s[i];
    }
  }
  if (threadIdx.x == 0 && shift && (!SHARED || blockIdx.y == 0)) shift[blockIdx.x] = xm;
}

// Layout of the task tables in the caller's work buffer: the series
// table, then (256-byte aligned) the task list.
size_t rw_task_offset(int32_t nlat) { return ((size_t)nlat * sizeof(RwLattice) + 255) / 256 * 256; }
size_t rw_work_bytes(int32_t nlat, int32_t ntask) {
  return rw_task_offset(nlat) + (size_t)ntask * sizeof(RwTask);
}

bool finite_nonneg(double v) { return std::isfinite(v) && v >= 0.0; }

// (U4, <E>/N, <|M|>/N) from one set of the five sums.
void quantities(const double* S, double N, double* q) {
  const double m2 = S[2] / S[0];
  const double m4 = S[3] / S[0];
  q[0] = 1.0 - m4 / (3.0 * m2 * m2);
  q[1] = S[4] / (S[0] * N);
  q[2] = S[1] / (S[0] * N);
}

// First k with d_k < 0 <= d_{k+1}, d = Ua - Ub; (T*, U*) or NaNs.
void crossing(const double* T, int K, const double* Ua, const double* Ub, double* Tx,
              double* Ux) {
  *Tx = *Ux = std::numeric_limits<double>::quiet_NaN();
  for (int k = 0; k + 1 < K; ++k) {
    const double d0 = Ua[k] - Ub[k], d1 = Ua[k + 1] - Ub[k + 1];
    if (d0 < 0.0 && 0.0 <= d1) {
      const double f = d0 / (d0 - d1);
      *Tx = T[k] + (T[k + 1] - T[k]) * f;
      *Ux = Ua[k] + (Ua[k + 1] - Ua[k]) * f;
      return;
    }
  }
}

// In-place radix-2 FFT of a (size a power of two) with the twiddles
// exp(-2 pi i k / n) taken from a table computed directly (no accumulated
// rotation), sign +1 for the inverse transform (unscaled).
void fft(std::vector<std::complex<double>>& a, int sign) {
  const size_t n = a.size();
  std::vector<std::complex<double>> tw(n / 2);
  for (size_t k = 0; k < n / 2; ++k) {
    const double ang = sign * 2.0 * M_PI * (double)k / (double)n;
    tw[k] = std::complex<double>(std::cos(ang), std::sin(ang));
  }
  for (size_t i = 1, j = 0; i < n; ++i) {
    size_t bit = n >> 1;
    for (; j & bit; bit >>= 1) j ^= bit;
    j ^= bit;
    if (i < j) std::swap(a[i], a[j]);
  }
  for (size_t len = 2; len <= n; len <<= 1) {
    const size_t half = len / 2, step = n / len;
    for (size_t i = 0; i < n; i += len)
      for (size_t j = 0; j < half; ++j) {
        const std::complex<double> u = a[i + j], v = a[i + j + half] * tw[j * step];
        a[i + j] = u + v;
        a[i + j + half] = u - v;
      }
  }
}

}  // namespace
}  // namespace ising

using namespace ising;

extern "C" {

size_t ising_reweight_work_bytes(int32_t nlat, int32_t ntask) {
  if (nlat < 1 || ntask < 1) return 0;
  return rw_work_bytes(nlat, ntask);
}

ising_status ising_reweight(int32_t nlat, const int64_t* const* dev_EM, const int64_t* n_sweeps,
                            const int64_t* discard, const double* beta0, int32_t ntask,
                            const int32_t* task_lattice, const double* task_beta,
                            int32_t nblocks, double* dev_sums, double* dev_shift,
                            void* dev_work, size_t work_bytes, void* hip_stream) {
  clear_error();
  if (nlat < 1 || ntask < 1 || !dev_EM || !n_sweeps || !discard || !beta0 || !task_lattice ||
      !task_beta || !dev_sums)
    return fail(ISING_EINVAL, "ising_reweight: bad arguments");
  if (!dev_work || ((uintptr_t)dev_work & 255) || work_bytes < rw_work_bytes(nlat, ntask))
    return fail(ISING_ENOMEM,
                "ising_reweight: needs a 256-byte aligned work buffer of %zu bytes (got %zu)",
                rw_work_bytes(nlat, ntask), dev_work ? work_bytes : (size_t)0);
  if (nblocks < 1 || nblocks > kRwMaxBlocks)
    return fail(ISING_EINVAL, "ising_reweight: nblocks must be in 1..%d", kRwMaxBlocks);
  std::vector<RwLattice> lat((size_t)nlat);
  for (int32_t i = 0; i < nlat; ++i) {
    if (!dev_EM[i] || discard[i] < 0 || n_sweeps[i] - discard[i] < nblocks ||
        !finite_nonneg(beta0[i]))
      return fail(ISING_EINVAL,
                  "ising_reweight: series %d needs a device pointer, 0 <= discard and at least "
                  "nblocks kept sweeps, and a finite beta0 >= 0",
                  i);
    lat[i] = RwLattice{dev_EM[i], n_sweeps[i], discard[i], beta0[i], 0, 0, 0};
  }
  std::vector<RwTask> tasks((size_t)ntask);
  for (int32_t k = 0; k < ntask; ++k) {
    if (task_lattice[k] < 0 || task_lattice[k] >= nlat || !finite_nonneg(task_beta[k]))
      return fail(ISING_EINVAL, "ising_reweight: task %d has a bad series index or beta", k);
    tasks[k] = RwTask{task_lattice[k], 0, task_beta[k]};
    lat[task_lattice[k]].used = 1;
  }
  const size_t off_task = rw_task_offset(nlat);
  const size_t bytes = rw_work_bytes(nlat, ntask);
  std::vector<char> img(bytes, 0);
  std::memcpy(img.data(), lat.data(), nlat * sizeof(RwLattice));
  std::memcpy(img.data() + off_task, tasks.data(), ntask * sizeof(RwTask));
  const hipStream_t st = (hipStream_t)hip_stream;
  hipError_t e = hipMemcpyAsync(dev_work, img.data(), bytes, hipMemcpyHostToDevice, st);
  if (e != hipSuccess) return hip_fail(e, "ising_reweight: table upload");
  // the host image must outlive the copy
  e = hipStreamSynchronize(st);
  if (e != hipSuccess) return hip_fail(e, "ising_reweight: table upload");
  hipLaunchKernelGGL(k_series_range, dim3(nlat), dim3(kRwThreads), 0, st, (RwLattice*)dev_work);
  e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "ising_reweight: launch");
  const RwLattice* dl = (const RwLattice*)dev_work;
  const RwTask* dt = (const RwTask*)((char*)dev_work + off_task);
  if (nblocks < 4 || (int64_t)ntask * nblocks <= kRwFewBlocks)
    hipLaunchKernelGGL(k_reweight<true>, dim3(ntask, nblocks), dim3(kRwThreads), 0, st, dl, dt,
                       nblocks, dev_sums, dev_shift);
  else
    hipLaunchKernelGGL(k_reweight<false>, dim3(ntask), dim3(kRwThreads), 0, st, dl, dt, nblocks,
                       dev_sums, dev_shift);
  e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "ising_reweight: launch");
  return ISING_OK;
}

ising_status ising_fss_moments(const double* sums, int32_t ntask, int32_t nblocks,
                               const int64_t* sites, double* est, double* err, double* u4_rep) {
  clear_error();
  if (!sums || !sites || !est || !err || ntask < 1 || nblocks < 2)
    return fail(ISING_EINVAL, "ising_fss_moments: bad arguments (nblocks >= 2)");
  std::vector<double> reps((size_t)nblocks * 3);
  for (int32_t k = 0; k < ntask; ++k) {
    const double* S = sums + (size_t)k * nblocks * 5;
    if (sites[k] < 1) return fail(ISING_EINVAL, "ising_fss_moments: sites[%d] < 1", k);
    const double N = (double)sites[k];
    double tot[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (int32_t b = 0; b < nblocks; ++b)
      for (int i = 0; i < 5; ++i) tot[i] += S[b * 5 + i];
    quantities(tot, N, est + 3 * (size_t)k);
    double mean[3] = {0.0, 0.0, 0.0};
    for (int32_t b = 0; b < nblocks; ++b) {
      double R[5];
      for (int i = 0; i < 5; ++i) R[i] = tot[i] - S[b * 5 + i];
      quantities(R, N, &reps[3 * (size_t)b]);
      for (int i = 0; i < 3; ++i) mean[i] += reps[3 * (size_t)b + i];
    }
    for (int i = 0; i < 3; ++i) mean[i] /= nblocks;
    for (int i = 0; i < 3; ++i) {
      double ss = 0.0;
      for (int32_t b = 0; b < nblocks; ++b) {
        const double dv = reps[3 * (size_t)b + i] - mean[i];
        ss += dv * dv;
      }
      err[3 * (size_t)k + i] = std::sqrt((double)(nblocks - 1) / nblocks * ss);
    }
    if (u4_rep)
      for (int32_t b = 0; b < nblocks; ++b) u4_rep[(size_t)k * nblocks + b] = reps[3 * (size_t)b];
  }
  return ISING_OK;
}

ising_status ising_autocorr_time(const double* x, int64_t n, double c, double* tau,
                                 int64_t* window) {
  clear_error();
  if (!x || n < 2 || !tau || !window || !(c > 0.0) || !std::isfinite(c))
    return fail(ISING_EINVAL, "ising_autocorr_time: bad arguments (n >= 2, c > 0)");
  if (n > (int64_t(1) << 28)) return fail(ISING_EINVAL, "ising_autocorr_time: n > 2^28");
  double mean = 0.0;
  for (int64_t i = 0; i < n; ++i) {
    if (!std::isfinite(x[i])) return fail(ISING_EINVAL, "ising_autocorr_time: x[%lld] not finite",
                                          (long long)i);
    mean += x[i];
  }
  mean /= (double)n;
  // sums S(t) = sum_{i < n - t} y_i y_{i+t} for all t at once: the inverse
  // transform of |FFT(y)|^2, zero-padded to avoid wrap-around
  size_t m = 1;
  while (m < 2 * (size_t)n) m <<= 1;
  std::vector<std::complex<double>> a(m, std::complex<double>(0.0, 0.0));
  double c0 = 0.0;
  for (int64_t i = 0; i < n; ++i) {
    const double y = x[i] - mean;
    a[i] = y;
    c0 += y * y;
  }
  c0 /= (double)n;
  if (c0 == 0.0) {
    *tau = 0.5;
    *window = 0;
    return ISING_OK;
  }
  fft(a, -1);
  for (size_t k = 0; k < m; ++k) a[k] = std::complex<double>(std::norm(a[k]), 0.0);
  fft(a, +1);
  double t = 0.5;
  for (int64_t W = 1; W <= n / 2; ++W) {
    t += a[W].real() / (double)m / (double)(n - W) / c0;
    if ((double)W >= c * t) {
      *tau = t;
      *window = W;
      return ISING_OK;
    }
  }
  *tau = t;
  *window = -1;
  return ISING_OK;
}

ising_status ising_binder_crossing(const double* T, int32_t K, const double* Ua,
                                   const double* Ub, const double* Ua_rep, const double* Ub_rep,
                                   int32_t nblocks, double* out) {
  clear_error();
  if (!T || !Ua || !Ub || !out || K < 2 || ((Ua_rep || Ub_rep) && (!Ua_rep || !Ub_rep)) ||
      ((Ua_rep != nullptr) && nblocks < 2))
    return fail(ISING_EINVAL, "ising_binder_crossing: bad arguments");
  for (int32_t k = 0; k + 1 < K; ++k)
    if (!(T[k] < T[k + 1])) return fail(ISING_EINVAL, "ising_binder_crossing: T not ascending");
  crossing(T, K, Ua, Ub, &out[0], &out[1]);
  const double nan = std::numeric_limits<double>::quiet_NaN();
  out[2] = out[3] = nan;
  if (!Ua_rep) return ISING_OK;
  std::vector<double> tx((size_t)nblocks), ux((size_t)nblocks);
  double mt = 0.0, mu = 0.0;
  for (int32_t b = 0; b < nblocks; ++b) {
    crossing(T, K, Ua_rep + (size_t)b * K, Ub_rep + (size_t)b * K, &tx[b], &ux[b]);
    if (std::isnan(tx[b])) return ISING_OK;
    mt += tx[b];
    mu += ux[b];
  }
  mt /= nblocks;
  mu /= nblocks;
  double st = 0.0, su = 0.0;
  for (int32_t b = 0; b < nblocks; ++b) {
    st += (tx[b] - mt) * (tx[b] - mt);
    su += (ux[b] - mu) * (ux[b] - mu);
  }
  out[2] = std::sqrt((double)(nblocks - 1) / nblocks * st);
  out[3] = std::sqrt((double)(nblocks - 1) / nblocks * su);
  return ISING_OK;
}

}  // extern "C"
