// Raw 3-D FFTs on device data (the FFT entry points of the paper's DKS usage
// example: data written to the device, a forward or inverse transform called
// on it, the result read back), on the same Stockham engine as the Poisson
// convolution: complex-to-complex forward and inverse, real-to-complex
// forward and complex-to-real inverse, every extent 2^a 3^b up to 4096,
// batched, unnormalised (inverse(forward(x)) = nx ny nz x).
//
// Layout: C-contiguous [batch][nz][ny][nx] (x fastest), interleaved complex.
// The real-to-complex transform keeps the nx/2 + 1 non-redundant x outputs
// per row ([batch][nz][ny][nx/2+1]); the complex-to-real inverse reads that
// layout.
//
// Passes: x is contiguous, so its tiles (W whole rows) are staged through LDS
// with linear, coalesced loads and stores; real rows of even length run on a
// complex transform of half the length.  y and z are strided: a tile is W
// adjacent columns (segments of 128 or 256 bytes; for z a plane's rows count
// as one), its first radix pass reads straight from HBM and its last pass
// writes straight to HBM.  Every pass reads its whole tile before it writes
// any of it, so in-place transforms are safe.

#ifndef DKS_FFT_RAW_PASSES_H
#define DKS_FFT_RAW_PASSES_H

#include "fft_engine.h"
#include "fft_raw_launch.h"

namespace dks {

// ---------------------------------------------------------------------------
// x: W rows per tile (row p of the tile holds element e at e / len, e mod len;
// the magic multipliers divide, len 1 aside).  kRowC2C: N complex in and out.  kRowR2C: N reals in
// (imaginary parts zero), the first N/2 + 1 outputs out.  kRowC2R: N/2 + 1
// complex in, completed to the full Hermitian row X[N - k] = conj X[k], the
// real parts of the inverse transform out.
// ---------------------------------------------------------------------------
// Values of its tile a lane stages; the length of a compile-time plan.
template <typename T, class SP> constexpr int row_regs() {
  if constexpr (SP::is_static) return (SP::N * SP::W + SP::TH - 1) / SP::TH;
  else return RegCfg<T>::EMAX;
}
template <class SP> constexpr int static_n() {
  if constexpr (SP::is_static) return SP::N;
  else return 1;
}
template <typename T, class SP, bool INV, int KIND>
__global__ __launch_bounds__((block_threads<T, SP>())) void k_fftr_rows(const void* __restrict__ in,
                                                                 void* __restrict__ out, long long nrows,
                                                                 const FFTPlan* __restrict__ P, int in_len,
                                                                 int out_len, unsigned magic_in,
                                                                 unsigned magic_out) {
  using C = typename Cplx<T>::type;
  constexpr int TH = block_threads<T, SP>();
  constexpr int KL = row_regs<T, SP>();
  extern __shared__ __align__(16) unsigned char smem[];
  C* lds = reinterpret_cast<C*>(smem);
  const int W = plan_W<SP>(P), LD = plan_LD<SP>(P), N = plan_N<SP>(P);
  const long long row0 = (long long)blockIdx.x * W;
  const int nvalid = (int)min((long long)W, nrows - row0);
  // element e of the tile's rows of `len` values -> its row
  auto row_of = [](int e, int len, unsigned magic, auto clen) {
    if constexpr (SP::is_static) return (int)((unsigned)e / (unsigned)decltype(clen)::value);
    else return len == 1 ? e : (int)__umulhi((unsigned)e, magic);
  };
  constexpr int NS = static_n<SP>();
  using InLen = std::integral_constant<int, KIND == kRowC2R ? NS / 2 + 1 : NS>;
  using OutLen = std::integral_constant<int, KIND == kRowR2C ? NS / 2 + 1 : NS>;
  {
    const int total = nvalid * in_len;
    if constexpr (KIND == kRowR2C) {
      const T* src = static_cast<const T*>(in) + row0 * in_len;
      T v[KL];
#pragma unroll
      for (int k = 0; k < KL; ++k) {
        const int e = (int)threadIdx.x + k * TH;
        v[k] = e < total ? src[e] : (T)0;
      }
#pragma unroll
      for (int k = 0; k < KL; ++k) {
        const int e = (int)threadIdx.x + k * TH;
        if (e < total) {
          const int p = row_of(e, in_len, magic_in, InLen{});
          const int x = e - p * in_len;
          lds[x * LD + p] = C{v[k], (T)0};
        }
      }
    } else {
      const C* src = static_cast<const C*>(in) + row0 * in_len;
      C v[KL];
#pragma unroll
      for (int k = 0; k < KL; ++k) {
        const int e = (int)threadIdx.x + k * TH;
        v[k] = e < total ? src[e] : C{0, 0};
      }
#pragma unroll
      for (int k = 0; k < KL; ++k) {
        const int e = (int)threadIdx.x + k * TH;
        if (e < total) {
          const int p = row_of(e, in_len, magic_in, InLen{});
          const int x = e - p * in_len;
          lds[x * LD + p] = v[k];
          if constexpr (KIND == kRowC2R) {
            if (x >= 1 && N - x > x) lds[(N - x) * LD + p] = C{v[k].x, -v[k].y};
          }
        }
      }
    }
  }
  __syncthreads();
  {
    auto lin = [&](int c, int idx, int) { return lds[idx * LD + c]; };
    auto lout = [&](auto RC, int c, int, int base, int Ns, C* vals, int) {
#pragma unroll
      for (int r = 0; r < RC.value; ++r) lds[(base + r * Ns) * LD + c] = vals[r];
    };
    run_any<T, INV, true, SP, 0>(lds, P, lin, lout);
  }
  __syncthreads();
  const int total = nvalid * out_len;
  if constexpr (KIND == kRowC2R) {
    T* dst = static_cast<T*>(out) + row0 * out_len;
#pragma unroll 4
    for (int e = (int)threadIdx.x; e < total; e += TH) {
      const int p = row_of(e, out_len, magic_out, OutLen{});
      const int x = e - p * out_len;
      dst[e] = lds[x * LD + p].x;
    }
  } else {
    C* dst = static_cast<C*>(out) + row0 * out_len;
#pragma unroll 4
    for (int e = (int)threadIdx.x; e < total; e += TH) {
      const int p = row_of(e, out_len, magic_out, OutLen{});
      const int x = e - p * out_len;
      dst[e] = lds[x * LD + p];
    }
  }
}

// ---------------------------------------------------------------------------
// x rows of real data of even length 2 N on a complex transform of length N
// (compile-time plans): a row's reals are the pairs z[m] = x[2m] + i x[2m+1].
// Forward: X[k] = (Z[k] + conj Z[N-k]) / 2 - i w^k (Z[k] - conj Z[N-k]) / 2,
// w = e^{-2 pi i / 2N}, k = 0 .. N.  Inverse: Z'[k] = (X[k] + conj X[N-k])
// + i w^-k (X[k] - conj X[N-k]), whose unnormalised inverse transform is
// 2N (x[2m] + i x[2m+1]); the imaginary parts of X[0] and X[N], which a real
// row does not have, are left out (they would only reach the imaginary part
// of the completed row's transform).  post: w^k, k = 0 .. N.  Half the tile
// and half the arithmetic of the full-length complex row, both sides of it
// contiguous in memory: 216 x 144 x 96 x 4 FP64 48 -> 39 us forward, 41 -> 35
// inverse.
// ---------------------------------------------------------------------------
template <typename T, class SP, bool INV>
__global__ __launch_bounds__((SP::TH)) void k_fftr_real_rows(const void* __restrict__ in, void* __restrict__ out,
                                                            long long nrows, const FFTPlan* __restrict__ P,
                                                            const typename Cplx<T>::type* __restrict__ post,
                                                            int pairs) {
  using C = typename Cplx<T>::type;
  constexpr int TH = SP::TH, N = SP::N, W = SP::W, LD = SP::LD;
  extern __shared__ __align__(16) unsigned char smem[];
  C* lds = reinterpret_cast<C*>(smem);
  C* lpost = lds + N * LD;
  const long long row0 = (long long)blockIdx.x * W;
  const int nvalid = (int)min((long long)W, nrows - row0);
  for (int k = (int)threadIdx.x; k <= N; k += TH) lpost[k] = post[k];
  auto lin = [&](int c, int idx, int) { return lds[idx * LD + c]; };
  auto lout = [&](auto RC, int c, int, int base, int Ns, C* vals, int) {
#pragma unroll
    for (int r = 0; r < RC.value; ++r) lds[(base + r * Ns) * LD + c] = vals[r];
  };
  constexpr int KP = (W * N + TH - 1) / TH;             // pairs per lane
  if constexpr (!INV) {
    const T* src = static_cast<const T*>(in) + row0 * (2 * N);
    const int total = nvalid * N;
    C v[KP];
#pragma unroll
    for (int i = 0; i < KP; ++i) {
      const int e = min((int)threadIdx.x + i * TH, total - 1);
      v[i] = pairs ? reinterpret_cast<const C*>(src)[e] : C{src[2 * e], src[2 * e + 1]};
    }
#pragma unroll
    for (int i = 0; i < KP; ++i) {
      const int e = (int)threadIdx.x + i * TH;
      if (e < total) lds[(int)((unsigned)e % (unsigned)N) * LD + (int)((unsigned)e / (unsigned)N)] = v[i];
    }
    __syncthreads();
    run_any<T, false, true, SP, 0>(lds, P, lin, lout);
    __syncthreads();
    C* dst = static_cast<C*>(out) + row0 * (N + 1);
    const int nout = nvalid * (N + 1);
    for (int e = (int)threadIdx.x; e < nout; e += TH) {
      const int p = (int)((unsigned)e / (unsigned)(N + 1)), k = e - p * (N + 1);
      const C zk = lds[(k == N ? 0 : k) * LD + p];
      C zc = lds[(k == 0 ? 0 : N - k) * LD + p];
      zc.y = -zc.y;
      const C s = cadd(zk, zc), d = csub(zk, zc);
      const C wd = cmul(lpost[k], d);
      dst[e] = C{(T)0.5 * (s.x + wd.y), (T)0.5 * (s.y - wd.x)};
    }
  } else {
    const C* src = static_cast<const C*>(in) + row0 * (N + 1);
    const int total = nvalid * N;
    C xk[KP], xc[KP];
#pragma unroll
    for (int i = 0; i < KP; ++i) {
      const int e = min((int)threadIdx.x + i * TH, total - 1);
      const int p = (int)((unsigned)e / (unsigned)N), k = e - p * N;
      xk[i] = src[p * (N + 1) + k];
      xc[i] = src[p * (N + 1) + N - k];
      if (k == 0) xk[i].y = xc[i].y = (T)0;
    }
    __syncthreads();                                    // lpost
#pragma unroll
    for (int i = 0; i < KP; ++i) {
      const int e = (int)threadIdx.x + i * TH;
      if (e < total) {
        const int p = (int)((unsigned)e / (unsigned)N), k = e - p * N;
        const C c{xc[i].x, -xc[i].y};
        const C s = cadd(xk[i], c), d = csub(xk[i], c);
        C w = lpost[k];
        w.y = -w.y;
        const C wd = cmul(w, d);
        lds[k * LD + p] = C{s.x - wd.y, s.y + wd.x};
      }
    }
    __syncthreads();
    run_any<T, true, true, SP, 0>(lds, P, lin, lout);
    __syncthreads();
    T* dst = static_cast<T*>(out) + row0 * (2 * N);
    for (int e = (int)threadIdx.x; e < total; e += TH) {
      const C z = lds[(int)((unsigned)e % (unsigned)N) * LD + (int)((unsigned)e / (unsigned)N)];
      if (pairs) {
        reinterpret_cast<C*>(dst)[e] = z;
      } else {
        dst[2 * e] = z.x;
        dst[2 * e + 1] = z.y;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// y or z: pencils of N elements S apart, W adjacent columns per tile.  Block
// b covers column tile b mod ntile of pencil group o = b / ntile, whose first
// element is (o / d1) s1 + (o mod d1) s2.
// ---------------------------------------------------------------------------
template <typename T, class SP, bool INV>
__global__ __launch_bounds__((block_threads<T, SP>())) void k_fftr_cols(const typename Cplx<T>::type* in,
                                                                 typename Cplx<T>::type* out, int ncols,
                                                                 int ntile, size_t S, int d1, size_t s1,
                                                                 size_t s2, const FFTPlan* __restrict__ P) {
  using C = typename Cplx<T>::type;
  using Off = OffT<SP>;
  extern __shared__ __align__(16) unsigned char smem[];
  C* lds = reinterpret_cast<C*>(smem);
  const int W = plan_W<SP>(P);
  const unsigned b = blockIdx.x;
  const unsigned o = b / (unsigned)ntile;
  const int tile = (int)(b - o * (unsigned)ntile);
  const unsigned o1 = o / (unsigned)d1, o2 = o - o1 * (unsigned)d1;
  const size_t base = (size_t)o1 * s1 + (size_t)o2 * s2 + (size_t)tile * W;
  const int ncol = min(W, ncols - tile * W);
  const C* src = in + base;
  C* dst = out + base;
  const Off st = (Off)S;
  auto rd = [&](int c, int idx, int) { return c < ncol ? src[(Off)idx * st + (Off)c] : C{0, 0}; };
  auto wr = [&](auto RC, int c, int, int bs, int Ns, C* vals, int) {
    if (c < ncol) {
#pragma unroll
      for (int r = 0; r < RC.value; ++r) dst[(Off)(bs + r * Ns) * st + (Off)c] = vals[r];
    }
  };
  run_any<T, INV, true, SP, 0>(lds, P, rd, wr);
}

template <typename T, bool INV, int KIND>
hipError_t launch_rows(const void* in, void* out, long long nrows, const PlanRef& P, int in_len, int out_len,
                              hipStream_t s) {
  const long long nblk = (nrows + P.host.W - 1) / P.host.W;
  if (nblk > 0x7fffffffLL) return hipErrorInvalidValue;
  const bool ok = with_row_plan<T>(P.host, [&](auto sp) {
    hipLaunchKernelGGL((k_fftr_rows<T, decltype(sp), INV, KIND>), dim3((unsigned)nblk),
                       dim3(block_threads<T, decltype(sp)>()), lds_bytes<T>(P.host), s, in, out, nrows, P.dev, in_len, out_len, magic_of(in_len),
                       magic_of(out_len));
  });
  return ok ? hipGetLastError() : hipErrorInvalidValue;
}

// Real rows of even length on the half-length plan P (real_rows_half).
template <typename T, bool INV>
hipError_t launch_real_rows(const void* in, void* out, long long nrows, const PlanRef& P, const void* post,
                            hipStream_t s) {
  using C = typename Cplx<T>::type;
  const long long nblk = (nrows + P.host.W - 1) / P.host.W;
  if (nblk > 0x7fffffffLL) return hipErrorInvalidValue;
  const int pairs = reinterpret_cast<uintptr_t>(INV ? out : in) % sizeof(C) == 0;
  bool ok = false;
  with_row_plan<T>(P.host, [&](auto sp) {
    using SP = decltype(sp);
    if constexpr (SP::is_static) {
      hipLaunchKernelGGL((k_fftr_real_rows<T, SP, INV>), dim3((unsigned)nblk), dim3(SP::TH),
                         lds_bytes<T>(P.host) + (size_t)(SP::N + 1) * sizeof(C), s, in, out, nrows, P.dev,
                         (const C*)post, pairs);
      ok = true;
    }
  });
  return ok ? hipGetLastError() : hipErrorInvalidValue;
}

template <typename T, bool INV>
hipError_t launch_cols(const void* in, void* out, int ncols, size_t S, int nouter, int d1, size_t s1,
                              size_t s2, size_t elems, const PlanRef& P, hipStream_t s) {
  using C = typename Cplx<T>::type;
  const int ntile = (ncols + P.host.W - 1) / P.host.W;
  const long long nblk = (long long)ntile * nouter;
  if (nblk > 0x7fffffffLL) return hipErrorInvalidValue;
  // 32-bit offsets inside a pencil tile when the whole array is addressable with them
  const bool off32 = cols_fit32(elems);
  const bool ok = with_col_plan<T>(P.host, [&](auto sp) {
    hipLaunchKernelGGL((k_fftr_cols<T, decltype(sp), INV>), dim3((unsigned)nblk),
                       dim3(block_threads<T, decltype(sp)>()), lds_bytes<T>(P.host), s, (const C*)in, (C*)out, ncols, ntile, S, d1, s1, s2, P.dev);
  }, off32);
  return ok ? hipGetLastError() : hipErrorInvalidValue;
}

}  // namespace dks

#endif  // DKS_FFT_RAW_PASSES_H
