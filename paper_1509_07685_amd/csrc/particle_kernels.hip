// Particle <-> mesh kernels of the PM step: bounding box of the bunch (the
// particle-fitted mesh of the PM section), per-solve geometry in FP64,
// cloud-in-cell deposit and gather (the "NGP, CIC, TSI" interpolation of the
// OPAL structure figure), and the central-difference field (its D-operators).

#include <math.h>

#include <type_traits>

#include "dks_internal.h"

namespace dks {

template <typename T> struct Vec4;
template <> struct Vec4<float> { using type = float4; };
template <> struct Vec4<double> { using type = double4; };

// Cell coordinate (x - x0) * (1/h) with two correctly rounded operations and
// no contraction, so the in/out and cell decisions are reproducible.
__device__ __forceinline__ float cell_coord(float x, float x0, float ih) {
  return __fmul_rn(__fsub_rn(x, x0), ih);
}
__device__ __forceinline__ double cell_coord(double x, double x0, double ih) {
  return __dmul_rn(__dsub_rn(x, x0), ih);
}

__device__ __forceinline__ const Geometry* geo_at(const Geometry* base, size_t stride, int b) {
  return reinterpret_cast<const Geometry*>(reinterpret_cast<const char*>(base) + (size_t)b * stride);
}

// ---------------------------------------------------------------------------
// Bounding box, stage 1: each block reduces a contiguous share of the
// particles of batch element blockIdx.y to (min x, min y, min z, max x, max y,
// max z) and writes it to its partial slot.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void k_bbox(ElemBatch eb, double* partial, size_t partial_stride) {
  const int b = blockIdx.y;
  const dks_particle_set e = eb.at(b);
  const T* p[3] = {(const T*)e.x, (const T*)e.y, (const T*)e.z};
  const int64_t n = eb.n(e);
  T lo[3], hi[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    lo[d] = INFINITY;
    hi[d] = -INFINITY;
  }
  int64_t start, end;
  chunk_of(n, blockIdx.x, gridDim.x, &start, &end);
  for_each_particle<T>(p[0], p[1], p[2], start, end, [&](T x, T y, T z, int64_t) {
    lo[0] = fmin(lo[0], x);
    hi[0] = fmax(hi[0], x);
    lo[1] = fmin(lo[1], y);
    hi[1] = fmax(hi[1], y);
    lo[2] = fmin(lo[2], z);
    hi[2] = fmax(hi[2], z);
  });
  __shared__ T red[6][256];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    red[d][threadIdx.x] = lo[d];
    red[3 + d][threadIdx.x] = hi[d];
  }
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        red[d][threadIdx.x] = fmin(red[d][threadIdx.x], red[d][threadIdx.x + s]);
        red[3 + d][threadIdx.x] = fmax(red[3 + d][threadIdx.x], red[3 + d][threadIdx.x + s]);
      }
    }
    __syncthreads();
  }
  if (threadIdx.x < 6)
    partial[(size_t)b * partial_stride + (size_t)blockIdx.x * 6 + threadIdx.x] = (double)red[threadIdx.x][0];
}

// ---------------------------------------------------------------------------
// Geometry of each batch element (one block per element): reduce the bbox
// partials, fit h and the origin, and derive every FP64 factor of the solve.
// The block also clears the out-of-mesh counter.  The whole is one chain of latencies in front of the step: the partials are
// reduced by shuffles, and lane d derives the values of axis d, so that the
// divisions of the three axes run side by side.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void geometry_of(int b, const double* partial, size_t partial_stride, Geometry* geo,
                                            size_t geo_stride, const GeoArgs& a, const ElemBatch& eb) {
#pragma clang fp contract(off)
  const dks_particle_set e = eb.at(b);
  Geometry* g = reinterpret_cast<Geometry*>(reinterpret_cast<char*>(geo) + (size_t)b * geo_stride);
  __shared__ double red[4][6];
  double v[6];                              // minima, then negated maxima
#pragma unroll
  for (int d = 0; d < 6; ++d) v[d] = INFINITY;
  if (a.fitted) {
    const double* pp = partial + (size_t)b * partial_stride;
    for (int i = threadIdx.x; i < a.nblocks; i += blockDim.x) {
#pragma unroll
      for (int d = 0; d < 6; ++d) v[d] = fmin(v[d], d < 3 ? pp[i * 6 + d] : -pp[i * 6 + d]);
    }
  }
  if (a.fitted) {
#pragma unroll
    for (int d = 0; d < 6; ++d) {
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) v[d] = fmin(v[d], __shfl_xor(v[d], o, 64));
      if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][d] = v[d];
    }
  }
  __syncthreads();
  if (threadIdx.x >= 3) return;
  const int d = (int)threadIdx.x;
  auto axis = [&](const double (&x)[3]) { return d == 0 ? x[0] : d == 1 ? x[1] : x[2]; };
  double h, origin;
  if (a.fitted) {
    const int n = d == 0 ? a.n[0] : d == 1 ? a.n[1] : a.n[2];
    const bool empty = eb.n(e) <= 0;
    const double lo = empty ? 0.0 : fmin(fmin(red[0][d], red[1][d]), fmin(red[2][d], red[3][d]));
    const double hi = empty ? 0.0 : -fmin(fmin(red[0][3 + d], red[1][3 + d]), fmin(red[2][3 + d], red[3][3 + d]));
    const double w = (hi - lo) / (double)(n - 3);
    h = fmax(fmax(fmax(0.0, __shfl(w, 0, 64)), __shfl(w, 1, 64)), __shfl(w, 2, 64));
    if (!(h > 0.0)) h = 1.0;
    origin = 0.5 * (lo + hi) - 0.5 * (double)(n - 1) * h;
  } else {
    h = axis(a.h);
    origin = axis(a.origin);
  }
  const double inv_h = 1.0 / h, grad = -1.0 / (2.0 * h);
  g->h[d] = h;
  g->origin[d] = origin;
  g->inv_h[d] = inv_h;
  g->grad_coef[d] = grad;
  g->origin_f[d] = (float)origin;
  g->inv_h_f[d] = (float)inv_h;
  g->grad_coef_f[d] = (float)grad;
  const double coulomb = 1.0 / (4.0 * M_PI * kEps0);
  if (d == 0) {
    double scale;
    if (a.mode == 0) scale = coulomb;                              // rho given in C/m^3
    else if (a.fitted) scale = coulomb * e.q / h;                  // spectrum built for h = 1 m
    else scale = coulomb * e.q / (a.h[0] * a.h[1] * a.h[2]);       // rho = q W / V
    g->conv_scale = scale;
    g->conv_scale_f = (float)scale;
  } else if (d == 1) {
    g->n_outside = 0;
  } else if (e.n_outside) {
    *e.n_outside = 0;
  }
}

__global__ __launch_bounds__(256) void k_geometry(const double* partial, size_t partial_stride,
                                                  Geometry* geo, size_t geo_stride, GeoArgs a,
                                                  ElemBatch eb) {
  geometry_of(blockIdx.x, partial, partial_stride, geo, geo_stride, a, eb);
}

// The geometry of element blockIdx.y (by workgroup 0 of the row) and the
// zero fills of that element's tile counters and deposit mesh (by every
// workgroup of the row): one launch for steps that do not depend on each
// other.
__global__ __launch_bounds__(256) void k_geometry_zero(const double* partial, size_t partial_stride,
                                                       Geometry* geo, size_t geo_stride, GeoArgs a,
                                                       ElemBatch eb, void* zbase, size_t zstride, size_t zbytes) {
  if (blockIdx.x == 0) geometry_of(blockIdx.y, partial, partial_stride, geo, geo_stride, a, eb);
  unsigned* z = reinterpret_cast<unsigned*>(reinterpret_cast<char*>(geo) + (size_t)blockIdx.y * geo_stride + a.zero_off);
  for (int i = (int)(blockIdx.x * blockDim.x + threadIdx.x); i < a.zero_len; i += (int)(gridDim.x * blockDim.x)) z[i] = 0u;
  char* p = reinterpret_cast<char*>(zbase) + (size_t)blockIdx.y * zstride;
  const size_t n16 = zbytes / 16;
  uint4* q = reinterpret_cast<uint4*>(p);
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x)
    q[i] = make_uint4(0, 0, 0, 0);
  const size_t tail = zbytes - n16 * 16;
  if (blockIdx.x == 0 && threadIdx.x < tail) p[n16 * 16 + threadIdx.x] = 0;
}

// rho = W * q / V for the deposit-only entry point (factor formed in FP64).
template <typename T>
__global__ __launch_bounds__(256) void k_weights_to_density(const T* W, T* rho, size_t n, const Geometry* g,
                                                            double q) {
  const double f = q / (g->h[0] * g->h[1] * g->h[2]);
  const T ft = (T)f;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    rho[i] = W[i] * ft;
}

// ---------------------------------------------------------------------------
// Central-difference field from phi with its ghost layer: E_d = -(phi(+e_d)
// - phi(-e_d)) / (2 h_d) on the physical nodes, written [3][nz][ny][nx].
// ---------------------------------------------------------------------------
// Bound by the stores (three meshes out for one in).  V nodes of a row per
// lane, 16 bytes of each component, with streaming stores; V = 1 where rows or
// outputs are not multiples of 16 bytes.  256^3 FP32, 270 MB: 48 us (5.6 TB/s);
// 73 with V = 1 and 61 with V = 4 and plain stores, which fill L2 and the
// last-level cache with a field that nothing reads next.
template <typename T, int V>
__global__ __launch_bounds__(256) void k_gradient(const T* __restrict__ phi, T* __restrict__ out,
                                                  const Geometry* g, MeshDims m) {
  typedef T VT __attribute__((ext_vector_type(V)));
  const int z = blockIdx.y;
  const int nx = m.nx, ny = m.ny, nz = m.nz, nv = nx / V;
  const int i2 = blockIdx.x * blockDim.x + threadIdx.x;    // V nodes of plane z
  if (i2 >= nv * ny) return;
  const int y = i2 / nv, x = (i2 - y * nv) * V;
  const T cx = Geo<T>::grad(g, 0), cy = Geo<T>::grad(g, 1), cz = Geo<T>::grad(g, 2);
  const size_t py = (size_t)nx + 2, pz = (size_t)(nx + 2) * (ny + 2);
  const T* c = phi + ((size_t)(z + 1) * pz + (size_t)(y + 1) * py + (size_t)(x + 1));
  // rows of phi start anywhere: vectors of element alignment
  auto row = [](const T* p) {
    VT v;
    __builtin_memcpy(&v, p, sizeof(VT));
    return v;
  };
  const VT mid = row(c), yp = row(c + py), ym = row(c - py), zp = row(c + pz), zm = row(c - pz);
  const T left = c[-1], right = c[V];
  VT ex, ey, ez;
#pragma unroll
  for (int k = 0; k < V; ++k) {
    ex[k] = cx * ((k + 1 < V ? mid[k + 1 < V ? k + 1 : 0] : right) - (k > 0 ? mid[k > 0 ? k - 1 : 0] : left));
    ey[k] = cy * (yp[k] - ym[k]);
    ez[k] = cz * (zp[k] - zm[k]);
  }
  const size_t i = ((size_t)z * ny + y) * nx + x, total = (size_t)nx * ny * nz;
  __builtin_nontemporal_store(ex, reinterpret_cast<VT*>(out + i));
  __builtin_nontemporal_store(ey, reinterpret_cast<VT*>(out + total + i));
  __builtin_nontemporal_store(ez, reinterpret_cast<VT*>(out + 2 * total + i));
}

// ---------------------------------------------------------------------------
// CIC gather of a [3][nz][ny][nx] mesh field at unsorted particles (the
// stand-alone gather entry point).  Outside particles receive 0.
// ---------------------------------------------------------------------------
template <typename T, int SCH>
__global__ __launch_bounds__(256) void k_gather(const T* __restrict__ E, const T* __restrict__ px,
                                                const T* __restrict__ py, const T* __restrict__ pz,
                                                T* __restrict__ qx, T* __restrict__ qy, T* __restrict__ qz,
                                                int64_t n, const Geometry* g, MeshDims m) {
  constexpr int WD = Scheme<SCH>::width;
  const T ox = Geo<T>::origin(g, 0), oy = Geo<T>::origin(g, 1), oz = Geo<T>::origin(g, 2);
  const T ix = Geo<T>::inv_h(g, 0), iy = Geo<T>::inv_h(g, 1), iz = Geo<T>::inv_h(g, 2);
  const int nx = m.nx, ny = m.ny, nz = m.nz;
  const size_t total = (size_t)nx * ny * nz;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    T wx[WD], wy[WD], wz[WD];
    int kx, ky, kz;
    // every axis is evaluated (its node and weights are set either way)
    const bool inx = axis_stencil<T, SCH>(cell_coord(px[i], ox, ix), nx, kx, wx);
    const bool iny = axis_stencil<T, SCH>(cell_coord(py[i], oy, iy), ny, ky, wy);
    const bool inz = axis_stencil<T, SCH>(cell_coord(pz[i], oz, iz), nz, kz, wz);
    const bool in = inx && iny && inz;
    T ax = 0, ay = 0, az = 0;
    if (in) {
      const int bx = kx + Scheme<SCH>::lo, by = ky + Scheme<SCH>::lo, bz = kz + Scheme<SCH>::lo;
#pragma unroll
      for (int cz = 0; cz < WD; ++cz)
#pragma unroll
        for (int cy = 0; cy < WD; ++cy)
#pragma unroll
          for (int cx = 0; cx < WD; ++cx) {
            const size_t node = ((size_t)(bz + cz) * ny + (by + cy)) * nx + (bx + cx);
            const T wgt = wz[cz] * wy[cy] * wx[cx];
            ax += wgt * E[node];
            ay += wgt * E[total + node];
            az += wgt * E[2 * total + node];
          }
    }
    qx[i] = ax;
    qy[i] = ay;
    qz[i] = az;
  }
}

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------
static inline unsigned grid_for(int64_t n, unsigned cap) {
  const int64_t b = (n + 255) / 256;
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(b, cap));
}

template <typename T>
hipError_t launch_bbox(const ElemBatch& eb, int batch, double* partial, size_t partial_stride, int* nblocks_out,
                       hipStream_t s) {
  // 2048 particles and more per workgroup: the fit reads every partial
  const unsigned nb = (unsigned)std::max<int64_t>(1, std::min<int64_t>((eb.max_np + 2047) / 2048, kBboxBlocks));
  *nblocks_out = (int)nb;
  hipLaunchKernelGGL(k_bbox<T>, dim3(nb, batch), dim3(256), 0, s, eb, partial, partial_stride);
  return hipGetLastError();
}

hipError_t launch_geometry(const double* partial, size_t partial_stride, Geometry* geo, size_t geo_stride,
                           const GeoArgs& a, const ElemBatch& eb, int batch, hipStream_t s) {
  hipLaunchKernelGGL(k_geometry, dim3(batch), dim3(256), 0, s, partial, partial_stride, geo, geo_stride, a, eb);
  return hipGetLastError();
}

hipError_t launch_geometry_zero(const double* partial, size_t partial_stride, Geometry* geo, size_t geo_stride,
                                const GeoArgs& a, const ElemBatch& eb, int batch, void* zbase, size_t zstride,
                                size_t zbytes, hipStream_t s) {
  const unsigned nb = grid_for((int64_t)(zbytes / 16 + 1), 8192);
  hipLaunchKernelGGL(k_geometry_zero, dim3(nb, batch), dim3(256), 0, s, partial, partial_stride, geo, geo_stride, a,
                     eb, zbase, zstride, zbytes);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_weights_to_density(const void* W, void* rho, size_t n, const Geometry* g, double q,
                                     hipStream_t s) {
  hipLaunchKernelGGL(k_weights_to_density<T>, dim3(grid_for((int64_t)n, 8192)), dim3(256), 0, s, (const T*)W,
                     (T*)rho, n, g, q);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_gradient(const void* phi, void* out, const Geometry* g, const MeshDims& m, hipStream_t s) {
  constexpr int V = 16 / (int)sizeof(T);
  const auto go = [&](auto kernel, int v) {
    const unsigned gx = (unsigned)(((int64_t)(m.nx / v) * m.ny + 255) / 256);
    hipLaunchKernelGGL(kernel, dim3(gx, m.nz), dim3(256), 0, s, (const T*)phi, (T*)out, g, m);
  };
  // 16-byte stores need rows (and with them the three components) of whole
  // vectors; 256^3 FP32: 48 us against 73
  if (m.nx % V == 0 && (reinterpret_cast<uintptr_t>(out) & 15u) == 0) go(k_gradient<T, V>, V);
  else go(k_gradient<T, 1>, 1);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_gather(const void* E, const void* x, const void* y, const void* z, void* ex, void* ey, void* ez,
                         int64_t n, const Geometry* g, const MeshDims& m, int scheme, hipStream_t s) {
  if (n == 0) return hipSuccess;
  auto go = [&](auto sc) {
    hipLaunchKernelGGL((k_gather<T, decltype(sc)::value>), dim3(grid_for(n, 65535u * 4)), dim3(256), 0, s,
                       (const T*)E, (const T*)x, (const T*)y, (const T*)z, (T*)ex, (T*)ey, (T*)ez, n, g, m);
  };
  if (scheme == kSchemeNGP) go(std::integral_constant<int, kSchemeNGP>{});
  else if (scheme == kSchemeTSC) go(std::integral_constant<int, kSchemeTSC>{});
  else go(std::integral_constant<int, kSchemeCIC>{});
  return hipGetLastError();
}

#define DKS_INSTANTIATE(T)                                                                                   \
  template hipError_t launch_bbox<T>(const ElemBatch&, int, double*, size_t, int*, hipStream_t);           \
  template hipError_t launch_weights_to_density<T>(const void*, void*, size_t, const Geometry*, double,      \
                                                   hipStream_t);                                             \
  template hipError_t launch_gradient<T>(const void*, void*, const Geometry*, const MeshDims&, hipStream_t); \
  template hipError_t launch_gather<T>(const void*, const void*, const void*, const void*, void*, void*,     \
                                       void*, int64_t, const Geometry*, const MeshDims&, int, hipStream_t);
DKS_INSTANTIATE(float)
DKS_INSTANTIATE(double)
#undef DKS_INSTANTIATE

}  // namespace dks
