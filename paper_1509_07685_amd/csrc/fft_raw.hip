// Raw 3-D FFTs on device data: plans and the C ABI (include/dks_fft.h).  The
// passes are in fft_raw_passes.h.

#include <cstring>
#include <new>
#include <vector>

#include "dks_fft.h"
#include "fft_engine.h"
#include "fft_plan_check.h"
#include "fft_raw_launch.h"

namespace dks {
template <typename T> hipError_t launch_twiddle_pass(void*, int, int, hipStream_t);
template <typename T> hipError_t launch_twiddle_line(void*, int, int, hipStream_t);
hipError_t launch_store_plans(const FFTPlan* four, FFTPlan* dev, hipStream_t s);
}  // namespace dks

using namespace dks;

// A raw FFT plan: three axis plans (x rows, y and z columns), their twiddle
// tables and device copies in the caller's workspace, plus the complex
// scratch of the complex-to-real inverse.
struct dks_fft_plan_s {
  int n[3];
  int batch;
  dks_fft_kind kind;
  dks_dtype dtype;
  size_t csize;
  FFTPlanHost pl[3];
  bool half;          // real rows on the half-length x plan
  size_t off_plans, off_tw[3], off_post, off_tmp, tmp_bytes, ws_total;
  char* ws;
  size_t ws_bytes;
  bool prepared;
};

namespace {

inline size_t al256(size_t v) { return (v + 255) & ~(size_t)255; }

bool is_23(int N) {
  if (N < 1) return false;
  while (N % 2 == 0) N /= 2;
  while (N % 3 == 0) N /= 3;
  return N == 1;
}

std::vector<int> radix_order(int N, bool fixed) {
  const RadixList l = static_radices(N);
  if (fixed && l.n > 0) return std::vector<int>(l.r, l.r + l.n);
  int a = 0, b = 0;
  while (N % 2 == 0) { N /= 2; ++a; }
  while (N % 3 == 0) { N /= 3; ++b; }
  std::vector<int> r;
  while (a >= 3) { r.push_back(8); a -= 3; }
  if (a == 2) r.push_back(4);
  if (a == 1) r.push_back(2);
  for (int i = 0; i < b; ++i) r.push_back(3);
  return r;
}

// fixed: the compile-time kernels run this axis where they know its length.
void make_axis(FFTPlanHost& P, int N, int W, int LD, bool fixed) {
  std::memset(&P, 0, sizeof(P));
  const std::vector<int> R = radix_order(N, fixed);
  P.dev.N = N;
  P.dev.npass = (int)R.size();
  P.dev.W = W;
  int lw = 0;
  while ((1 << lw) < W) ++lw;
  P.dev.logW = lw;
  P.dev.LD = LD;
  int Ns = 1, off = 0;
  for (size_t p = 0; p < R.size(); ++p) {
    P.dev.R[p] = R[p];
    P.dev.Ns[p] = Ns;
    P.dev.magic[p] = Ns >= 2 ? (unsigned)(((1ull << 32) + (unsigned long long)Ns - 1) / (unsigned long long)Ns) : 0u;
    P.dev.tw_off[p] = off;
    if (p > 0) off += Ns * (R[p] - 1);
    Ns *= R[p];
  }
  P.tw_count = off;
}

size_t row_len_complex(const dks_fft_plan_s* p) { return p->kind == DKS_FFT_R2C ? (size_t)(p->n[0] / 2 + 1) : (size_t)p->n[0]; }

PlanRef axis_ref(const dks_fft_plan_s* p, int a) {
  PlanRef r;
  r.host = p->pl[a].dev;
  r.host.tw = p->ws + p->off_tw[a];
  r.dev = reinterpret_cast<const FFTPlan*>(p->ws + p->off_plans) + a;
  return r;
}

// y then z column passes on the complex array `cur` (in place), or from
// `src` into `cur` for the first pass that runs.
template <typename T, bool INV>
dks_status run_cols(const dks_fft_plan_s* p, const void* src, void* cur, hipStream_t st) {
  const int nx = p->n[0], ny = p->n[1], nz = p->n[2];
  const size_t L = row_len_complex(p);
  const size_t elems = L * ny * nz * p->batch;
  const void* from = src;
  if (ny > 1) {
    if (launch_cols<T, INV>(from, cur, (int)L, L, nz * p->batch, 1, L * ny, 0, elems, axis_ref(p, 1), st) !=
        hipSuccess)
      return DKS_EHIP;
    from = cur;
  }
  if (nz > 1) {
    // a plane's rows are contiguous: its ny L elements are one run of columns
    // (no ragged tile per row, and every tile aligned like the plane)
    if (launch_cols<T, INV>(from, cur, (int)(L * ny), L * ny, p->batch, 1, L * ny * nz, 0, elems, axis_ref(p, 2),
                            st) != hipSuccess)
      return DKS_EHIP;
    from = cur;
  }
  (void)nx;
  if (from != cur) {   // no column pass ran: move the data
    if (hipMemcpyAsync(cur, src, elems * p->csize, hipMemcpyDeviceToDevice, st) != hipSuccess) return DKS_EHIP;
  }
  return DKS_OK;
}

template <typename T>
dks_status execute(const dks_fft_plan_s* p, const void* in, void* out, bool inverse, hipStream_t st) {
  const long long rows = (long long)p->n[1] * p->n[2] * p->batch;
  const int nx = p->n[0];
  const int nh = nx / 2 + 1;
  if (p->kind == DKS_FFT_C2C) {
    const hipError_t e = inverse ? launch_rows<T, true, kRowC2C>(in, out, rows, axis_ref(p, 0), nx, nx, st)
                                 : launch_rows<T, false, kRowC2C>(in, out, rows, axis_ref(p, 0), nx, nx, st);
    if (e != hipSuccess) return DKS_EHIP;
    return inverse ? run_cols<T, true>(p, out, out, st) : run_cols<T, false>(p, out, out, st);
  }
  if (!inverse) {
    const hipError_t e = p->half ? launch_real_rows<T, false>(in, out, rows, axis_ref(p, 0), p->ws + p->off_post, st)
                                 : launch_rows<T, false, kRowR2C>(in, out, rows, axis_ref(p, 0), nx, nh, st);
    if (e != hipSuccess) return DKS_EHIP;
    return run_cols<T, false>(p, out, out, st);
  }
  // complex-to-real: columns from the input into the scratch, then the rows
  const bool cols = p->n[1] > 1 || p->n[2] > 1;
  const void* rows_in = in;
  if (cols) {
    char* tmp = p->ws + p->off_tmp;
    const dks_status r = run_cols<T, true>(p, in, tmp, st);
    if (r != DKS_OK) return r;
    rows_in = tmp;
  }
  const hipError_t e = p->half ? launch_real_rows<T, true>(rows_in, out, rows, axis_ref(p, 0), p->ws + p->off_post, st)
                               : launch_rows<T, true, kRowC2R>(rows_in, out, rows, axis_ref(p, 0), nh, nx, st);
  return e == hipSuccess ? DKS_OK : DKS_EHIP;
}

}  // namespace

extern "C" {

dks_status dks_fft_plan(int nx, int ny, int nz, int batch, dks_fft_kind kind, dks_dtype dtype,
                        dks_fft_plan_t* out) {
  if (!out) return DKS_EINVAL;
  *out = nullptr;
  if (dtype != DKS_F32 && dtype != DKS_F64) return DKS_EINVAL;
  if (kind != DKS_FFT_C2C && kind != DKS_FFT_R2C) return DKS_EINVAL;
  if (batch < 1 || nx < 1 || ny < 1 || nz < 1) return DKS_EINVAL;
  const int ns[3] = {nx, ny, nz};
  for (int n : ns)
    if (n > kMaxLength || !is_23(n)) return DKS_EUNSUPPORTED;
  // every pass's workgroup count must fit a 1-D grid (checked again at launch)
  if ((double)ny * nz * batch > 2147483647.0) return DKS_EINVAL;
  dks_fft_plan_s* p = new (std::nothrow) dks_fft_plan_s;
  if (!p) return DKS_ENOMEM;
  std::memset(p, 0, sizeof(*p));
  p->n[0] = nx;
  p->n[1] = ny;
  p->n[2] = nz;
  p->batch = batch;
  p->kind = kind;
  p->dtype = dtype;
  p->csize = dtype == DKS_F32 ? 8 : 16;
  const int c = (int)p->csize;
  const int wmax = 128 / c;
  // x: padded row tiles (unpadded single rows when even one padded row does not fit)
  p->half = kind == DKS_FFT_R2C && real_rows_half(nx);
  const int mx = p->half ? nx / 2 : nx;
  const int Wx = row_width(mx, c, wmax);
  const bool padded = (size_t)mx * (Wx + 1) * c <= (size_t)kLdsBytes;
  make_axis(p->pl[0], mx, Wx, padded ? Wx + 1 : Wx, true);
  const size_t elems = row_len_complex(p) * (size_t)ny * nz * batch;
  const bool fit = cols_fit32(elems);
  for (int a = 1; a < 3; ++a) {
    int W = wide_columns(ns[a], elems, c, row_len_complex(p) * c) ? 2 * wmax : wmax;
    while (W > 1 && (size_t)ns[a] * W * c > (size_t)kLdsBytes) W >>= 1;
    make_axis(p->pl[a], ns[a], W, W, fit);
  }
  size_t off = 0;
  p->off_plans = off;
  off = al256(off + 4 * sizeof(FFTPlan));
  for (int a = 0; a < 3; ++a) {
    p->off_tw[a] = off;
    off = al256(off + (size_t)p->pl[a].tw_count * p->csize + 16);
  }
  p->off_post = off;
  if (p->half) off = al256(off + (size_t)(mx + 1) * p->csize);
  // the pass kernels' invariants: rows staged through EMAX registers per
  // thread (N values per row at most), columns read straight from memory
  {
    EngineLimits L;
    L.threads = dtype == DKS_F32 ? RegCfg<float>::THREADS : RegCfg<double>::THREADS;
    L.emax = dtype == DKS_F32 ? RegCfg<float>::EMAX : RegCfg<double>::EMAX;
    L.max_length = kMaxLength;
    L.max_pass = kMaxPass;
    L.lds_hw = kLdsHardware;
    bool fixed[3] = {false, false, false};     // the launchers' choice
    for (int a = 0; a < 3; ++a) {
      const auto see = [&](auto sp) { fixed[a] = decltype(sp)::is_static; };
      const auto pick = [&](auto t) {
        using T = decltype(t);
        if (a == 0) with_row_plan<T>(p->pl[0].dev, see);
        else with_col_plan<T>(p->pl[a].dev, see, fit);
      };
      if (dtype == DKS_F32) pick(0.0f);
      else pick(0.0);
    }
    int v = fft_plan_violation(p->pl[0].dev, L, p->csize, mx, L.emax, p->half ? (size_t)(mx + 1) * p->csize : 0,
                               fixed[0]);
    for (int a = 1; a < 3 && v == kPlanOk; ++a) v = fft_plan_violation(p->pl[a].dev, L, p->csize, 0, 0, 0, fixed[a]);
    // half-length rows have compile-time kernels only
    if (p->half && !fixed[0]) v = kPlanStructure;
    if (v != kPlanOk) {
      delete p;
      return DKS_EUNSUPPORTED;
    }
  }
  p->off_tmp = off;
  p->tmp_bytes = kind == DKS_FFT_R2C ? al256((size_t)(nx / 2 + 1) * ny * nz * batch * p->csize) : 0;
  p->ws_total = p->off_tmp + p->tmp_bytes;
  *out = p;
  return DKS_OK;
}

dks_status dks_fft_workspace_bytes(dks_fft_plan_t p, size_t* bytes) {
  if (!p || !bytes) return DKS_EINVAL;
  *bytes = p->ws_total;
  return DKS_OK;
}

dks_status dks_fft_set_workspace(dks_fft_plan_t p, void* ws, size_t bytes) {
  if (!p) return DKS_EINVAL;
  if (!ws || bytes < p->ws_total || (reinterpret_cast<uintptr_t>(ws) & 255) != 0) return DKS_EWORKSPACE;
  p->ws = static_cast<char*>(ws);
  p->ws_bytes = bytes;
  p->prepared = false;
  return DKS_OK;
}

dks_status dks_fft_prepare(dks_fft_plan_t p, dks_stream_t stream) {
  if (!p) return DKS_EINVAL;
  if (!p->ws) return DKS_EWORKSPACE;
  const hipStream_t st = static_cast<hipStream_t>(stream);
  for (int a = 0; a < 3; ++a) {
    const FFTPlan& f = p->pl[a].dev;
    for (int q = 1; q < f.npass; ++q) {
      void* dst = p->ws + p->off_tw[a] + (size_t)f.tw_off[q] * p->csize;
      const hipError_t e = p->dtype == DKS_F32 ? launch_twiddle_pass<float>(dst, f.Ns[q], f.R[q], st)
                                               : launch_twiddle_pass<double>(dst, f.Ns[q], f.R[q], st);
      if (e != hipSuccess) return DKS_EHIP;
    }
  }
  if (p->half) {
    void* post = p->ws + p->off_post;
    const hipError_t e = p->dtype == DKS_F32 ? launch_twiddle_line<float>(post, p->n[0], p->n[0] / 2 + 1, st)
                                             : launch_twiddle_line<double>(post, p->n[0], p->n[0] / 2 + 1, st);
    if (e != hipSuccess) return DKS_EHIP;
  }
  FFTPlan four[4];
  for (int a = 0; a < 3; ++a) four[a] = axis_ref(p, a).host;
  four[3] = four[2];
  if (launch_store_plans(four, reinterpret_cast<FFTPlan*>(p->ws + p->off_plans), st) != hipSuccess) return DKS_EHIP;
  p->prepared = true;
  return DKS_OK;
}

static dks_status fft_exec(dks_fft_plan_t p, const void* in, void* out, bool inverse, dks_stream_t stream) {
  if (!p || !in || !out) return DKS_EINVAL;
  if (p->kind == DKS_FFT_R2C && in == out) return DKS_EINVAL;
  if (!p->ws) return DKS_EWORKSPACE;
  if (!p->prepared) return DKS_ESTATE;
  const hipStream_t st = static_cast<hipStream_t>(stream);
  return p->dtype == DKS_F32 ? execute<float>(p, in, out, inverse, st) : execute<double>(p, in, out, inverse, st);
}

dks_status dks_fft_forward(dks_fft_plan_t p, const void* in, void* out, dks_stream_t stream) {
  return fft_exec(p, in, out, false, stream);
}

dks_status dks_fft_inverse(dks_fft_plan_t p, const void* in, void* out, dks_stream_t stream) {
  return fft_exec(p, in, out, true, stream);
}

dks_status dks_fft_destroy(dks_fft_plan_t p) {
  if (!p) return DKS_EINVAL;
  delete p;
  return DKS_OK;
}

}  // extern "C"
