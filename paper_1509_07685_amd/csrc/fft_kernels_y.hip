// The y passes of the convolution.
#include "fft_conv.h"

namespace dks {

#define DKS_INSTANTIATE(T) \
  template hipError_t launch_fft_y_fwd<T>(const void*, void*, size_t, const MeshDims&, const PlanRef&, int, int, int, \
                                          size_t, hipStream_t);                                                        \
  template hipError_t launch_fft_y_inv<T>(const void*, void*, size_t, const MeshDims&, const PlanRef&, int, int, int, \
                                          hipStream_t);
DKS_INSTANTIATE(float)
DKS_INSTANTIATE(double)
#undef DKS_INSTANTIATE

}  // namespace dks
