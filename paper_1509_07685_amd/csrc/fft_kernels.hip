// The x passes of the convolution, and the device copies of the plans.
#include "fft_conv.h"

namespace dks {

// Copies the host-built plans into device memory (kernel arguments are
// copied at launch, so this is safe inside stream capture).
__global__ void k_store_plans(FFTPlan a, FFTPlan b, FFTPlan c, FFTPlan d, FFTPlan* out) {
  if (threadIdx.x == 0) {
    out[0] = a;
    out[1] = b;
    out[2] = c;
    out[3] = d;
  }
}

hipError_t launch_store_plans(const FFTPlan* four, FFTPlan* dev, hipStream_t s) {
  hipLaunchKernelGGL(k_store_plans, dim3(1), dim3(64), 0, s, four[0], four[1], four[2], four[3], dev);
  return hipGetLastError();
}

#define DKS_INSTANTIATE(T) \
  template hipError_t launch_fft_x_fwd<T>(const void*, size_t, bool, void*, size_t, const MeshDims&,           \
                                          const PlanRef&, const void*, int, hipStream_t);                      \
  template hipError_t launch_fft_x_inv<T>(const void*, size_t, void*, size_t, const ElemBatch&, const MeshDims&, \
                                          const PlanRef&, const void*, int, hipStream_t);
DKS_INSTANTIATE(float)
DKS_INSTANTIATE(double)
#undef DKS_INSTANTIATE

}  // namespace dks
