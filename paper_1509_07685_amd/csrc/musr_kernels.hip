// Chi-square and maximum-likelihood evaluation of muon-spin-rotation positron
// histograms on the device (section "Parameter Fitting with Minuit2": the
// positron histogram and asymmetry equations give the model, the chi-square
// and log-likelihood equations the statistic).  The histograms stay resident;
// a call brings only the parameter vector and produces one FP64 number.
//
// One fused kernel per call: every workgroup takes 256 consecutive time
// bins of a group of up to 16 detectors and a run of parameter sets,
// evaluates the model, accumulates the statistic in FP64, reduces it across
// the workgroup in a fixed order and stores a partial per set; a
// one-workgroup-per-set kernel then adds the partials in index order, so a
// result is bitwise reproducible.  (A last-workgroup-done counter in the
// first kernel would need an agent-scope release and acquire per workgroup,
// i.e. an L2 write-back and invalidate each, which measured slower than the
// second launch.)

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>

#include <hip/hip_runtime.h>

#include "dks_musr.h"
#include "musr_math.h"

namespace dks {
namespace musr {

constexpr int kMaxDet = 32;
constexpr int kMaxSets = 1024;
constexpr int kThreads = 256;
constexpr int kGroup = 16;      // most detectors per workgroup: their counts stay in registers
constexpr int kRun = 8;         // most parameter sets per workgroup: 36 KB of LDS, four workgroups per CU
constexpr double kTauMu = 2.1969811;                         // muon lifetime, us
constexpr double kGammaMu = 6.283185307179586 * 0.01355388094;   // rad / (us G)

// Parameters of one evaluation, passed by value (kernel argument): sigma, B
// and per detector N0, Nbkg, A0 N0 cos(phi), A0 N0 sin(phi).
struct Params {
  double sigma, B;
  double det[4 * kMaxDet];
};

// Sum over the wavefront in a fixed order (xor shuffles).
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Sum over the workgroup in a fixed order: within each wavefront by xor
// shuffles, then the four wavefront sums in order.
__device__ __forceinline__ double block_sum(double v, double* lds) {
  v = wave_sum(v);
  const int w = (int)threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) lds[w] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < kThreads / 64; ++i) s += lds[i];
  __syncthreads();
  return s;
}

// The statistic's term as it is defined.
template <int STAT>
__device__ __forceinline__ double term(double d, double N) {
  if constexpr (STAT == DKS_MUSR_CHISQ) {
    const double r = d - N;
    return d > 0.0 ? r * r / d : r * r;
  } else {
    return d > 0.0 ? (N - d) + d * log(d / N) : N - d;
  }
}

// Counts of 0 or with a high word between these, ratios N / d likewise and
// squares (d - N)^2 up to the higher one take the fast terms below; anything
// else (negative, not finite, out of range) takes term().
constexpr unsigned kLowWord = 0x03f00000u, kHighWord = 0x7bf00000u;   // of 2^-960 and 2^960

struct DeviceOps {
  static __device__ __forceinline__ double estimate(double d) { return __builtin_amdgcn_rcp(d); }
  // a b + c with a constant c kept in scalar registers (the compiler's
  // two-address form copies a constant into the destination before every step
  // of a polynomial: a sixth of the batch's instructions).
  static __device__ __forceinline__ double fma_const(double a, double b, double c) {
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(c));
    return r;
  }
};

// grid: (time-bin blocks, detector groups, runs of `run` sets); partial:
// [sets][gx * gy].  A thread owns one time bin t = n dt and every detector of
// its group for each set of its run: the counts d and their reciprocals are
// formed once for all sets, and per set exp(-t/tau - (sigma t)^2 / 2) and
// cos/sin of the precession angle gamma B t once for all detectors, whose
// counts follow by cos(w t + phi_j) = cos(w t) cos(phi_j) - sin(w t)
// sin(phi_j) in three multiply-adds.  Both quotients, (d - N)^2 / d and N / d
// (log(d / N) = -log(N / d)), are products with 1 / d corrected by their exact
// remainder, so they are rounded like divisions; a plain product would carry
// the reciprocal's rounding, which is the same in every bin with that count.
// Bound by FP64 vector issue: 133 sets of 16 x 206250 bins took 1.55 ms
// (log-likelihood) when every term divided twice and ran the library
// logarithm, 0.72 ms now.
template <int STAT, bool DEV>
__global__ __launch_bounds__(kThreads, DEV && STAT == DKS_MUSR_MLE ? 3 : 4) void k_musr_eval(const double* __restrict__ data, long long n_bins,
                                                           double dt, Params prm, const double* __restrict__ dprm,
                                                           int nparam, int n_det, int dg, int nsets, int run,
                                                           double* __restrict__ partial) {
  // per set of the run and detector of the group: N0, Nbkg, A0 N0 cos(phi), A0 N0 sin(phi)
  __shared__ double cst[DEV ? kRun * kGroup * 4 : 1];
  __shared__ double sums[DEV ? kRun : 1][kThreads / 64];
  __shared__ double2 uv[DEV ? kRun : 1][DEV ? kThreads : 1];   // a lane's own entries: cos and sin parts per set
  const int tid = (int)threadIdx.x;
  const int set0 = blockIdx.z * run;
  const int ns = DEV ? min(run, nsets - set0) : 1;
  const int j0 = blockIdx.y * dg;
  const int nj = min(dg, n_det - j0);
  const long long n = (long long)blockIdx.x * kThreads + tid;
  const bool live = n < n_bins;
  const double* col = data + (size_t)j0 * n_bins + (live ? n : n_bins - 1);
  const double t = (double)n * dt;
  const double a = -t / kTauMu;
  auto damped = [&](double sigma, double B) {
    const double EG = exp(a - 0.5 * (sigma * t) * (sigma * t));
    double sw, cw;
    sincos(kGammaMu * B * t, &sw, &cw);
    return make_double2(EG * cw, -EG * sw);
  };
  double d[kGroup], rd[kGroup];
  double2 own;
  if constexpr (DEV) {
    // before the counts are loaded: their registers would be held through
    // the sine's argument reduction, which needs many
    for (int i = tid; i < ns * kGroup; i += kThreads) {
      const int s = i / kGroup, j = i % kGroup;
      if (j < nj) {
        const double* q = dprm + (size_t)(set0 + s) * nparam + 2 + 4 * (j0 + j);
        double sp, cp;
        sincos(q[3], &sp, &cp);
        double* c = cst + i * 4;
        c[0] = q[0];
        c[1] = q[1];
        c[2] = q[2] * q[0] * cp;
        c[3] = q[2] * q[0] * sp;
      }
    }
#pragma unroll 1
    for (int s = 0; s < ns; ++s) {
      const double* q = dprm + (size_t)(set0 + s) * nparam;
      uv[s][tid] = damped(q[0], q[1]);
    }
  }
#pragma unroll
  for (int j = 0; j < kGroup; ++j) d[j] = j < nj ? col[(size_t)j * n_bins] : 1.0;
  if constexpr (!DEV) own = damped(prm.sigma, prm.B);
  const double E = exp(a);
  bool odd = false;          // some count out of the fast terms' range
#pragma unroll
  for (int j = 0; j < kGroup; ++j) {
    odd |= (d[j] != 0.0) & ((unsigned)__double2hiint(d[j]) - kLowWord > kHighWord - kLowWord);
    rd[j] = d[j] > 0.0 ? recip<DeviceOps>(d[j]) : 0.5;         // quotient(n, 0, 1/2) = n
  }
  if constexpr (DEV) __syncthreads();
#pragma unroll 1
  for (int s = 0; s < ns; ++s) {
    if constexpr (DEV) own = uv[s][tid];
    const double u = own.x, v = own.y;
    // constants of detector j of the group: LDS, or scalar loads of the kernel argument
    auto model = [&](int j) {
      if constexpr (DEV) {
        const double* c = cst + (s * kGroup + j) * 4;
        return fma(c[0], E, fma(c[2], u, fma(c[3], v, c[1])));
      } else {
        const double* c = prm.det + 4 * (j0 + j);
        return fma(c[0], E, fma(c[2], u, fma(c[3], v, c[1])));
      }
    };
    double acc = 0.0;
    // the largest high word of a quotient N / d, as a distance from the least
    // one allowed, or of a square
    constexpr unsigned least = STAT == DKS_MUSR_MLE ? kLowWord : 0u;
    unsigned far = 0;
    auto one = [&](int j) {
      const double N = model(j);
      if constexpr (STAT == DKS_MUSR_CHISQ) {
        const double r = d[j] - N, r2 = r * r;
        far = max(far, (unsigned)__double2hiint(r2));
        acc += quotient(r2, d[j], rd[j]);
      } else {
        // d = 0 weighs its logarithm with 0
        const double x = quotient(N, d[j], rd[j]);
        far = max(far, (unsigned)__double2hiint(x) - least);
        acc += fma(-d[j], log_normal<DeviceOps>(x), N - d[j]);
      }
    };
    // four detectors at a time, their chains interleaved, then the rest
#pragma unroll
    for (int jb = 0; jb < kGroup; jb += 4) {
      if (jb + 4 <= nj) {
#pragma unroll
        for (int j = jb; j < jb + 4; ++j) one(j);
      } else {
#pragma unroll
        for (int j = jb; j < jb + 3; ++j)
          if (j < nj) one(j);
      }
    }
    if (odd || far > kHighWord - least) {
      acc = 0.0;
#pragma unroll 1
      for (int j = 0; j < nj; ++j) {
        acc += term<STAT>(col[(size_t)j * n_bins], model(j));
      }
    }
    const double w = wave_sum(live ? acc : 0.0);
    if ((tid & 63) == 0) sums[s][tid >> 6] = w;
  }
  __syncthreads();
  if (tid < ns) {
    double w = 0.0;
    for (int i = 0; i < kThreads / 64; ++i) w += sums[tid][i];
    partial[(size_t)(set0 + tid) * gridDim.x * gridDim.y + blockIdx.y * gridDim.x + blockIdx.x] = w;
  }
}

// One workgroup per set: the set's partials added in index order.
template <int STAT>
__global__ __launch_bounds__(kThreads) void k_musr_final(const double* __restrict__ partial, int nblk,
                                                         double* __restrict__ result) {
  __shared__ double red[kThreads / 64];
  const double* part = partial + (size_t)blockIdx.x * nblk;
  double v = 0.0;
  for (int i = (int)threadIdx.x; i < nblk; i += kThreads) v += part[i];
  const double tot = block_sum(v, red);
  if (threadIdx.x == 0) result[blockIdx.x] = STAT == DKS_MUSR_MLE ? 2.0 * tot : tot;
}

}  // namespace musr
}  // namespace dks

using namespace dks::musr;

struct dks_musr_plan_s {
  int n_det;
  long long n_bins;
  double dt;
  int max_sets;
  int bx;                 // time-bin workgroups
  int dg, gy;             // detectors per group, groups
  size_t ws_total;
  char* ws;
  const double* data;
  bool prepared;
};

namespace {

inline size_t al256(size_t v) { return (v + 255) & ~(size_t)255; }

template <int STAT, bool DEV>
hipError_t launch(const dks_musr_plan_s* p, const Params& prm, const double* dprm, int nsets, double* result,
                  hipStream_t st) {
  double* partial = reinterpret_cast<double*>(p->ws);
  // Batches: as many detectors per group as leave about four workgroups per
  // CU (the plan's groups are those of one set), and runs of sets, which
  // share the counts' reciprocals, as long as leave twice that.
  int dg = p->dg, gy = p->gy, run = 1;
  if (DEV) {
    const long long per_group = (long long)p->bx * nsets;
    gy = (int)std::min<long long>(gy, std::max<long long>((p->n_det + kGroup - 1) / kGroup, (1024 + per_group - 1) / per_group));
    dg = (p->n_det + gy - 1) / gy;
    gy = (p->n_det + dg - 1) / dg;
    const int want = (int)std::min<long long>(kRun, std::max<long long>(1, per_group * gy / 2048));
    const int runs = (nsets + want - 1) / want;
    run = (nsets + runs - 1) / runs;
  }
  hipLaunchKernelGGL((k_musr_eval<STAT, DEV>), dim3(p->bx, gy, (nsets + run - 1) / run), dim3(kThreads), 0, st,
                     p->data, p->n_bins, p->dt, prm, dprm, 2 + 4 * p->n_det, p->n_det, dg, nsets, run, partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_musr_final<STAT>), dim3(nsets), dim3(kThreads), 0, st, partial, p->bx * gy, result);
  return hipGetLastError();
}

dks_status run(const dks_musr_plan_s* p, dks_musr_stat stat, const Params& prm, const double* dprm, int nsets,
               double* result, hipStream_t st) {
  hipError_t e;
  if (stat == DKS_MUSR_CHISQ)
    e = dprm ? launch<DKS_MUSR_CHISQ, true>(p, prm, dprm, nsets, result, st)
             : launch<DKS_MUSR_CHISQ, false>(p, prm, dprm, nsets, result, st);
  else
    e = dprm ? launch<DKS_MUSR_MLE, true>(p, prm, dprm, nsets, result, st)
             : launch<DKS_MUSR_MLE, false>(p, prm, dprm, nsets, result, st);
  return e == hipSuccess ? DKS_OK : DKS_EHIP;
}

dks_status ready(const dks_musr_plan_s* p) {
  if (!p->ws) return DKS_EWORKSPACE;
  if (!p->prepared || !p->data) return DKS_ESTATE;
  return DKS_OK;
}

}  // namespace

extern "C" {

dks_status dks_musr_plan(int n_det, int64_t n_bins, double dt, int max_sets, dks_musr_plan_t* out) {
  if (!out) return DKS_EINVAL;
  *out = nullptr;
  if (n_det < 1 || n_det > kMaxDet || n_bins < 1 || n_bins > 0x7fffffffLL) return DKS_EINVAL;
  if (!(dt > 0.0) || !std::isfinite(dt) || max_sets < 1 || max_sets > kMaxSets) return DKS_EINVAL;
  dks_musr_plan_s* p = new (std::nothrow) dks_musr_plan_s;
  if (!p) return DKS_ENOMEM;
  std::memset(p, 0, sizeof(*p));
  p->n_det = n_det;
  p->n_bins = n_bins;
  p->dt = dt;
  p->max_sets = max_sets;
  p->bx = (int)((n_bins + kThreads - 1) / kThreads);
  // share the per-bin transcendentals across as many detectors as a group
  // holds while keeping at least ~512 workgroups per set in flight
  const long long least = std::max<long long>((n_det + kGroup - 1) / kGroup, (512 + p->bx - 1) / p->bx);
  const int groups = (int)std::min<long long>(n_det, least);
  p->dg = (n_det + groups - 1) / groups;
  p->gy = (n_det + p->dg - 1) / p->dg;
  p->ws_total = al256((size_t)max_sets * p->bx * p->gy * sizeof(double));
  *out = p;
  return DKS_OK;
}

dks_status dks_musr_workspace_bytes(dks_musr_plan_t p, size_t* bytes) {
  if (!p || !bytes) return DKS_EINVAL;
  *bytes = p->ws_total;
  return DKS_OK;
}

dks_status dks_musr_set_workspace(dks_musr_plan_t p, void* ws, size_t bytes) {
  if (!p) return DKS_EINVAL;
  if (!ws || bytes < p->ws_total || (reinterpret_cast<uintptr_t>(ws) & 255) != 0) return DKS_EWORKSPACE;
  p->ws = static_cast<char*>(ws);
  p->prepared = false;
  return DKS_OK;
}

dks_status dks_musr_prepare(dks_musr_plan_t p, dks_stream_t stream) {
  (void)stream;
  if (!p) return DKS_EINVAL;
  if (!p->ws) return DKS_EWORKSPACE;
  p->prepared = true;   // the workspace holds only per-call partials: nothing to initialise
  return DKS_OK;
}

dks_status dks_musr_set_data(dks_musr_plan_t p, const double* data) {
  if (!p || !data) return DKS_EINVAL;
  p->data = data;
  return DKS_OK;
}

dks_status dks_musr_eval(dks_musr_plan_t p, dks_musr_stat stat, const double* params, double* result,
                         dks_stream_t stream) {
  if (!p || !params || !result || (stat != DKS_MUSR_CHISQ && stat != DKS_MUSR_MLE)) return DKS_EINVAL;
  const dks_status r = ready(p);
  if (r != DKS_OK) return r;
  Params prm;
  std::memset(&prm, 0, sizeof(prm));
  prm.sigma = params[0];
  prm.B = params[1];
  for (int j = 0; j < p->n_det; ++j) {
    const double* q = params + 2 + 4 * j;
    prm.det[4 * j] = q[0];
    prm.det[4 * j + 1] = q[1];
    double sp, cp;
    sincos(q[3], &sp, &cp);
    prm.det[4 * j + 2] = q[2] * q[0] * cp;
    prm.det[4 * j + 3] = q[2] * q[0] * sp;
  }
  return run(p, stat, prm, nullptr, 1, result, static_cast<hipStream_t>(stream));
}

dks_status dks_musr_eval_batch(dks_musr_plan_t p, dks_musr_stat stat, const double* params, int nsets,
                               double* results, dks_stream_t stream) {
  if (!p || !params || !results || (stat != DKS_MUSR_CHISQ && stat != DKS_MUSR_MLE)) return DKS_EINVAL;
  if (nsets < 1 || nsets > p->max_sets) return DKS_EINVAL;
  const dks_status r = ready(p);
  if (r != DKS_OK) return r;
  Params prm;
  std::memset(&prm, 0, sizeof(prm));
  return run(p, stat, prm, params, nsets, results, static_cast<hipStream_t>(stream));
}

dks_status dks_musr_destroy(dks_musr_plan_t p) {
  if (!p) return DKS_EINVAL;
  delete p;
  return DKS_OK;
}

}  // extern "C"
