// The z pass of the convolution in FP32.
#include "fft_conv.h"

namespace dks {

template hipError_t launch_fft_z_conv<float>(const void*, void*, size_t, const void*, const Geometry*, size_t, const MeshDims&,
                                         const PlanRef&, const PlanRef&, int, int, int, hipStream_t);

}  // namespace dks
