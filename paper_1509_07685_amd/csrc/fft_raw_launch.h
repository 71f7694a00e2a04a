// Launchers of the raw transforms' passes (fft_raw_passes.h, instantiated per
// dtype in fft_raw_f32.hip and fft_raw_f64.hip) and the rules plan creation
// shares with them.
#ifndef DKS_FFT_RAW_LAUNCH_H
#define DKS_FFT_RAW_LAUNCH_H

#include "fft_engine.h"

namespace dks {

enum RowKind { kRowC2C = 0, kRowR2C = 1, kRowC2R = 2 };

// Tile width of an x (row) tile: the widest power of two <= w whose padded
// tile (N (W + 1) complex values) fits the LDS budget.
constexpr int row_width(int N, int c, int w) { return (w > 1 && N * (w + 1) * c > kLdsBytes) ? row_width(N, c, w / 2) : w; }

// 32-bit offsets inside a pencil tile when the whole array is addressable with them.
inline bool cols_fit32(size_t elems) { return elems < 0x7fffffffULL; }

// Column tiles of 256 instead of 128 bytes per row, for lengths up to 256 (the
// tile then still takes at most 64 KiB) of arrays of 64 MiB and more: the
// segments of a strided pencil pass lie a row or a plane apart, and twice the
// run per segment raised the z pass of 512 x 512 x 256 FP32 from 3.7 to 4.8
// TB/s (290 -> 222 us) and the 216 x 144 x 96 x 4 FP64 columns from 50 and 49
// to 30 and 40 us.  Smaller arrays stay in the caches and want the larger
// number of tiles (96^3 FP64: 22.7 against 25.5 us for the three passes).
constexpr int kWideMaxLength = 256;
inline bool wide_columns(int N, size_t elems, size_t csize) {
  return N <= kWideMaxLength && static_radices(N).n > 0 && cols_fit32(elems) && elems * csize >= ((size_t)64 << 20);
}

// Real rows of even length whose half has compile-time kernels.
inline bool real_rows_half(int nx) { return nx % 2 == 0 && static_radices(nx / 2).n > 0; }

template <typename T, bool INV, int KIND>
hipError_t launch_rows(const void* in, void* out, long long nrows, const PlanRef& P, int in_len, int out_len,
                       hipStream_t s);
template <typename T, bool INV>
hipError_t launch_real_rows(const void* in, void* out, long long nrows, const PlanRef& P, const void* post,
                            hipStream_t s);
template <typename T, bool INV>
hipError_t launch_cols(const void* in, void* out, int ncols, size_t S, int nouter, int d1, size_t s1, size_t s2,
                       size_t elems, const PlanRef& P, hipStream_t s);

}  // namespace dks

#endif  // DKS_FFT_RAW_LAUNCH_H
