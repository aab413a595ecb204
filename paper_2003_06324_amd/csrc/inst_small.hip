// Kernel instantiations: small products, one 32x32 block per workgroup.
#include "gemm_launch.h"
namespace gemm_gfx950 {
GEMM_INSTANTIATE_SMALL(_Float16)
GEMM_INSTANTIATE_SMALL(__bf16)
GEMM_INSTANTIATE_SMALL(float)
}
