// Kernel instantiations: small products, one 32x32 (or 16x16) block per workgroup.
#include "gemm_launch.h"
namespace gemm_gfx950 {
GEMM_INSTANTIATE_SMALL(_Float16)
GEMM_INSTANTIATE_SMALL(__bf16)
GEMM_INSTANTIATE_SMALL(float)
template hipError_t launch_small16<float>(bool, bool, dim3, hipStream_t, const KernelArgs &);
}
