// Chi-square and maximum-likelihood evaluation of muon-spin-rotation positron
// histograms on the device (section "Parameter Fitting with Minuit2": the
// positron histogram and asymmetry equations give the model, the chi-square
// and log-likelihood equations the statistic).  The histograms stay resident;
// a call brings only the parameter vector and produces one FP64 number.
//
// One fused kernel per call: every workgroup takes 256 consecutive time
// bins of a group of 16 (or 4) detectors and a run of parameter sets,
// evaluates the model, accumulates the statistic in FP64, reduces it across
// the workgroup in a fixed order and stores a partial per set; a
// one-workgroup-per-set kernel then adds the partials in a fixed order, so a
// result is bitwise reproducible.  (A last-workgroup-done counter in the
// first kernel, with release and acquire fences around the partials, takes an
// L2 write-back and invalidate per workgroup, which measured slower than the
// second launch.)
//
// A set's result does not depend on how many sets are evaluated with it, or
// by which entry point: every sum is formed in one order, four detectors of a
// bin, over the 256 lanes, the fours of a sixteen, the sixteens of a block of
// bins, the blocks, wherever the launch's groups put the steps.

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
constexpr int kQuad = 4;        // detectors summed in one lane
constexpr int kGroup = 16;      // most detectors per workgroup: their counts stay in registers
constexpr int kQuads = kGroup / kQuad;
constexpr int kRun = 8;         // most parameter sets per workgroup: 38 KB of LDS, four workgroups per CU
constexpr double kTauMu = 2.1969811;                         // muon lifetime, us
constexpr double kGammaMu = 6.283185307179586 * 0.01355388094;   // rad / (us G)

// Parameters of one evaluation, passed by value (kernel argument).
struct Params {
  double sigma, B;
  double det[kMaxDet][4];   // N0, Nbkg, A0, phi
};

// The four values of q summed over the wavefront in a fixed order (xor
// shuffles), in 7 exchanges instead of 24: each half keeps two of the four
// values at the first step, each quarter one at the second.  Lane l returns
// the sum of value (l & 32 ? 1 : 0) + (l & 16 ? 2 : 0).
__device__ __forceinline__ double wave_sum4(const double (&q)[kQuads]) {
  static_assert(kQuads == 4, "two halving steps");
  const bool hi = threadIdx.x & 32, odd = threadIdx.x & 16;
  const double a = (hi ? q[1] : q[0]) + __shfl_xor(hi ? q[0] : q[1], 32, 64);
  const double b = (hi ? q[3] : q[2]) + __shfl_xor(hi ? q[2] : q[3], 32, 64);
  double v = (odd ? b : a) + __shfl_xor(odd ? a : b, 16, 64);
#pragma unroll
  for (int o = 8; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
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

// grid: (time-bin blocks, detector groups, runs of at most RUN sets); partial:
// [sets][groups][blocks].  A thread owns one time bin t = n dt and every
// detector of its group (G = kGroup, or kQuad where the blocks alone do not
// fill the chip) for each set of its run: the counts d and their reciprocals
// are formed once for all sets, and per set exp(-t/tau - (sigma t)^2 / 2) and
// cos/sin of the precession angle gamma B t once for all detectors, whose
// counts follow by cos(w t + phi_j) = cos(w t) cos(phi_j) - sin(w t)
// sin(phi_j) in three multiply-adds.  Both quotients, (d - N)^2 / d and N / d
// (log(d / N) = -log(N / d)), are products with 1 / d corrected by their exact
// remainder, so they are rounded like divisions.
// Bound by FP64 vector issue: 133 sets of 16 x 206250 bins took 1.55 ms
// (log-likelihood; chi-square 0.56) when every term divided twice and ran the
// library logarithm, 0.75 ms (0.30) now.  A single evaluation is bound by the
// latency of its one chain per lane and by the two launches (12.6 -> 12.0 us).
template <int STAT, bool DEV, int RUN, int G>
__global__ __launch_bounds__(kThreads, RUN > 1 && STAT == DKS_MUSR_MLE ? 3 : 4) void k_musr_eval(
    const double* __restrict__ data, long long n_bins, double dt, Params prm, const double* __restrict__ dprm,
    int nparam, int n_det, int dg, int nsets, int run, double* __restrict__ partial) {
  static_assert(DEV || RUN == 1, "one set by value");
  constexpr int Q = G / kQuad;
  // per set of the run and detector of the group: N0, Nbkg, A0 N0 cos(phi), A0 N0 sin(phi)
  __shared__ double cst[RUN * G * 4];
  __shared__ double sums[RUN][kQuads][kThreads / 64];
  __shared__ double2 uv[RUN > 1 ? RUN : 1][RUN > 1 ? kThreads : 1];   // a lane's own entries: cos and sin parts per set
  const int tid = (int)threadIdx.x;
  const int set0 = blockIdx.z * run;
  const int ns = RUN > 1 ? min(run, nsets - set0) : 1;
  const int j0 = blockIdx.y * dg;
  const int nj = min(dg, n_det - j0);
  const long long n = (long long)blockIdx.x * kThreads + tid;
  const bool live = n < n_bins;
  const double* col = data + (size_t)j0 * n_bins + (live ? n : n_bins - 1);
  const double t = (double)n * dt;
  const double a = -t / kTauMu;
  // (contractions written out: every instance rounds alike)
  auto damped = [&](double sigma, double B) {
    const double st = sigma * t;
    const double EG = exp(fma(-0.5 * st, st, a));
    double sw, cw;
    sincos(kGammaMu * B * t, &sw, &cw);
    return make_double2(EG * cw, -EG * sw);
  };
  auto constants = [&](int i, double N0, double Nb, double A0, double phi) {
    double sp, cp;
    sincos(phi, &sp, &cp);
    double* c = cst + i * 4;
    c[0] = N0;
    c[1] = Nb;
    c[2] = A0 * N0 * cp;
    c[3] = A0 * N0 * sp;
  };
  double d[G], rd[G];
  // (no load is conditional: a group's last detector is read again past its
  // end, so the compiler can wait for the constants below without waiting for
  // the counts)
  auto load = [&]() {
#pragma unroll
    for (int j = 0; j < G; ++j) d[j] = col[(size_t)min(j, nj - 1) * n_bins];
  };
  // one set: the constants are requested before the counts and formed, with
  // the lane's own factors, while those are on their way; a run's counts are
  // loaded after its sines: their registers would be held through the argument
  // reductions, which need many
  if constexpr (RUN == 1) {
    double q[4];
    if (tid < nj) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        q[k] = DEV ? dprm[(size_t)set0 * nparam + 2 + 4 * (j0 + tid) + k] : prm.det[j0 + tid][k];
    }
    load();
    if (tid < nj) constants(tid, q[0], q[1], q[2], q[3]);
  } else {
    for (int i = tid; i < ns * G; i += kThreads) {
      const int s = i / G, j = i % G;
      if (j < nj) {
        const double* q = dprm + (size_t)(set0 + s) * nparam + 2 + 4 * (j0 + j);
        constants(i, q[0], q[1], q[2], q[3]);
      }
    }
  }
  double2 own;
  if constexpr (RUN > 1) {
#pragma unroll 1
    for (int s = 0; s < ns; ++s) {
      const double* q = dprm + (size_t)(set0 + s) * nparam;
      uv[s][tid] = damped(q[0], q[1]);
    }
    load();
  } else if constexpr (DEV) {
    const double* q = dprm + (size_t)set0 * nparam;
    own = damped(q[0], q[1]);
  } else {
    own = damped(prm.sigma, prm.B);
  }
  const double E = exp(a);
  bool odd[Q] = {};          // per four detectors: some count out of the fast terms' range
#pragma unroll
  for (int j = 0; j < G; ++j) {
    odd[j / kQuad] |= (d[j] != 0.0) & ((unsigned)__double2hiint(d[j]) - kLowWord > kHighWord - kLowWord);
    rd[j] = d[j] > 0.0 ? recip<DeviceOps>(d[j]) : 0.5;         // quotient(n, 0, 1/2) = n
  }
  __syncthreads();
#pragma unroll 1
  for (int s = 0; s < ns; ++s) {
    if constexpr (RUN > 1) own = uv[s][tid];
    const double u = own.x, v = own.y;
    auto model = [&](int j) {
      const double* c = cst + (s * G + j) * 4;
      return fma(c[0], E, fma(c[2], u, fma(c[3], v, c[1])));
    };
    double acc[kQuads] = {0.0, 0.0, 0.0, 0.0};
    bool slow[Q], any = !live;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      // the largest high word of a quotient N / d, as a distance from the
      // least one allowed, or of a square
      constexpr unsigned least = STAT == DKS_MUSR_MLE ? kLowWord : 0u;
      unsigned far = 0;
      auto one = [&](int j) {
        const double N = model(j);
        if constexpr (STAT == DKS_MUSR_CHISQ) {
          const double r = d[j] - N, r2 = r * r;
          far = max(far, (unsigned)__double2hiint(r2));
          acc[q] += quotient(r2, d[j], rd[j]);
        } else {
          // d = 0 weighs its logarithm with 0
          const double x = quotient(N, d[j], rd[j]);
          far = max(far, (unsigned)__double2hiint(x) - least);
          acc[q] += fma(-d[j], log_normal<DeviceOps>(x), N - d[j]);
        }
      };
      const int jb = q * kQuad;
      // whole fours with their chains interleaved, then the rest
      if (jb + kQuad <= nj) {
#pragma unroll
        for (int j = jb; j < jb + kQuad; ++j) one(j);
      } else {
#pragma unroll
        for (int j = jb; j < jb + kQuad - 1; ++j)
          if (j < nj) one(j);
      }
      slow[q] = odd[q] | (far > kHighWord - least);
      any |= slow[q];
    }
    if (any) {
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        if (live && !slow[q]) continue;
        acc[q] = 0.0;
#pragma unroll 1
        for (int j = q * kQuad; live && j < min((q + 1) * kQuad, nj); ++j)
          acc[q] += term<STAT>(col[(size_t)j * n_bins], model(j));
      }
    }
    const double w = wave_sum4(acc);
    if ((tid & 15) == 0) sums[s][(tid >> 5 & 1) + (tid >> 4 & 1) * 2][tid >> 6] = w;
  }
  __syncthreads();
  if (tid < ns) {
    double w = 0.0;
    for (int q = 0; q * kQuad < nj; ++q) {
      const double* p = sums[tid][q];
      w += ((p[0] + p[1]) + p[2]) + p[3];
    }
    partial[((size_t)(set0 + tid) * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] = w;
  }
}

// One workgroup per set: the partials of its nblk blocks of bins, each block's
// gy groups added first (fours of detectors to sixteens, `per` of them, and
// these in order).  The sum over the blocks is carried in two words (each
// addition's exact rounding error beside it), because its few last additions
// round by far the most: the result's relative error over 160 sets of 16 x
// 206250 bins went from 9.0e-17 (chi-square) and 8.1e-17 (log-likelihood) rms to
// 5.7e-17 and 5.2e-17 for 0.6 us.
template <int STAT>
__global__ __launch_bounds__(kThreads) void k_musr_final(const double* __restrict__ partial, int nblk, int gy, int per,
                                                         double* __restrict__ result) {
  __shared__ double2 red[kThreads / 64];
  const double* part = partial + (size_t)blockIdx.x * nblk * gy;
  double2 v = make_double2(0.0, 0.0);
  auto add = [&](double hi, double lo) {
    const double s = v.x + hi, t = s - v.x;
    v = make_double2(s, v.y + lo + ((v.x - (s - t)) + (hi - t)));
  };
  for (int i = (int)threadIdx.x; i < nblk; i += kThreads) {
    double block = 0.0;
    for (int g = 0; g < gy; g += per) {
      double w = 0.0;
      for (int u = g; u < min(g + per, gy); ++u) w += part[(size_t)u * nblk + i];
      block += w;
    }
    add(block, 0.0);
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) add(__shfl_xor(v.x, o, 64), __shfl_xor(v.y, o, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    v = red[0];
    for (int i = 1; i < kThreads / 64; ++i) add(red[i].x, red[i].y);
    // (an infinite or undefined sum has no error beside it)
    const double tot = isfinite(v.x) ? v.x + v.y : v.x;
    result[blockIdx.x] = STAT == DKS_MUSR_MLE ? 2.0 * tot : tot;
  }
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
  size_t ws_total;
  char* ws;
  const double* data;
  bool prepared;
};

namespace {

inline size_t al256(size_t v) { return (v + 255) & ~(size_t)255; }

int groups_of(int n_det, int dg) { return (n_det + dg - 1) / dg; }

// Detectors per whole group: fours in as few groups of at most kGroup as hold
// them, spread evenly.
int group_size(int n_det) {
  const int quads = groups_of(n_det, kQuad), groups = groups_of(quads, kQuads);
  return (quads + groups - 1) / groups * kQuad;
}

// Groups of four detectors for a call of nsets sets: where a workgroup per
// block, whole group and set would leave some of the chip's 256 CUs without
// one (16 x 50000 bins, 196 blocks, log-likelihood: 11.2 us split; where there
// are enough, each group's own exponentials and sines cost more than they
// hide: 16 x 206250, 806 blocks, 16.2 us whole and 28 split).
constexpr int kSplitFill = 256;
bool split_groups(const dks_musr_plan_s* p, int nsets) {
  return (long long)p->bx * groups_of(p->n_det, group_size(p->n_det)) * nsets < kSplitFill;
}

constexpr int kRunFill = 1024;

template <int STAT, bool DEV>
hipError_t launch(const dks_musr_plan_s* p, const Params& prm, const double* dprm, int nsets, double* result,
                  hipStream_t st) {
  double* partial = reinterpret_cast<double*>(p->ws);
  const bool split = split_groups(p, nsets);
  const int whole = group_size(p->n_det), dg = split ? kQuad : whole, gy = groups_of(p->n_det, dg);
  // runs of sets, which share the counts' loads and reciprocals, as long as
  // leave four workgroups per CU (5 sets of 16 x 206250 bins: chi-square 24.5
  // us in one run of 806 workgroups, 25.6 in two, 27.6 one by one;
  // log-likelihood 46.7, 43.4 and 44.2)
  int run = 1;
  if (DEV && !split) {
    const int want = (int)std::min<long long>(kRun, std::max<long long>(1, (long long)p->bx * gy * nsets / kRunFill));
    const int runs = (nsets + want - 1) / want;
    run = (nsets + runs - 1) / runs;
  }
  const auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(p->bx, gy, (nsets + run - 1) / run), dim3(kThreads), 0, st, p->data, p->n_bins,
                       p->dt, prm, dprm, 2 + 4 * p->n_det, p->n_det, dg, nsets, run, partial);
  };
  if (split) {
    go(k_musr_eval<STAT, DEV, 1, kQuad>);
  } else if (DEV && run > 1) {
    if constexpr (DEV) go(k_musr_eval<STAT, true, kRun, kGroup>);
  } else {
    go(k_musr_eval<STAT, DEV, 1, kGroup>);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_musr_final<STAT>), dim3(nsets), dim3(kThreads), 0, st, partial, p->bx, gy,
                     split ? whole / kQuad : 1, result);
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
  // partials of the largest call, split or not
  size_t sets_split = 0;
  while ((int)sets_split < max_sets && split_groups(p, (int)sets_split + 1)) ++sets_split;
  p->ws_total = al256(std::max((size_t)max_sets * groups_of(n_det, group_size(n_det)), sets_split * groups_of(n_det, kQuad)) *
                      p->bx * sizeof(double));
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
  for (int j = 0; j < p->n_det; ++j)
    for (int q = 0; q < 4; ++q) prm.det[j][q] = params[2 + 4 * j + q];
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
