// The direct GEMM (gemm_direct.h) on tiled operands.
#include "gemm_direct.h"

bool sq_direct_gemm_launch_tiled(const GemmArgs& a, const DirectArgs& q, int mb, int nb, int nw, hipStream_t st)
{
    return direct_gemm_launch<true>(a, q, mb, nb, nw, st);
}
