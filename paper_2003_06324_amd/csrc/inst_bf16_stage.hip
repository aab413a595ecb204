// Kernel instantiations: bf16 operands, tiles for launches of at most one workgroup per CU.
#include "gemm_launch.h"
namespace gemm_gfx950 {
GEMM_INSTANTIATE_STAGE(__bf16, 64, 64, 6)
GEMM_INSTANTIATE_STAGE(__bf16, 64, 128, 5)
GEMM_INSTANTIATE_STAGE(__bf16, 128, 64, 5)
GEMM_INSTANTIATE_STAGE(__bf16, 128, 128, 4)
}
