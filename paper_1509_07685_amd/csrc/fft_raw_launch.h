// Launchers of the raw transforms' passes (fft_raw_passes.h, instantiated per
// dtype in fft_raw_f32.hip and fft_raw_f64.hip).
#ifndef DKS_FFT_RAW_LAUNCH_H
#define DKS_FFT_RAW_LAUNCH_H

#include "fft_engine.h"

namespace dks {

enum RowKind { kRowC2C = 0, kRowR2C = 1, kRowC2R = 2 };

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
