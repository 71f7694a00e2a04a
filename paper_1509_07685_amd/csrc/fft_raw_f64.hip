// The passes of the raw FP64 transforms.
#include "fft_raw_passes.h"

namespace dks {

#define DKS_ROWS(INV, KIND) \
  template hipError_t launch_rows<double, INV, KIND>(const void*, void*, long long, const PlanRef&, int, int, hipStream_t);
#define DKS_DIR(INV)                                                                                             \
  template hipError_t launch_real_rows<double, INV>(const void*, void*, long long, const PlanRef&, const void*, hipStream_t); \
  template hipError_t launch_cols<double, INV>(const void*, void*, int, size_t, int, int, size_t, size_t, size_t,    \
                                              const PlanRef&, hipStream_t);
DKS_ROWS(false, kRowC2C)
DKS_ROWS(true, kRowC2C)
DKS_ROWS(false, kRowR2C)
DKS_ROWS(true, kRowC2R)
DKS_DIR(false)
DKS_DIR(true)
#undef DKS_ROWS
#undef DKS_DIR

}  // namespace dks
