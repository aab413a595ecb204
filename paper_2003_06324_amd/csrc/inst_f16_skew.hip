// Kernel instantiations: f16 operands, tiles for launches of at most one workgroup per CU, rows that begin off the cache lines.
#include "gemm_launch.h"
namespace gemm_gfx950 {
GEMM_INSTANTIATE_SKEW(_Float16, 64, 64, 7)
GEMM_INSTANTIATE_SKEW(_Float16, 64, 128, 6)
GEMM_INSTANTIATE_SKEW(_Float16, 128, 64, 6)
GEMM_INSTANTIATE_SKEW(_Float16, 128, 128, 5)
}
