// The direct GEMM (gemm_direct.h) on row-major operands.
#include "gemm_direct.h"

bool sq_direct_gemm_launch_rows(const GemmArgs& a, const DirectArgs& q, int mb, int nb, int nw, hipStream_t st)
{
    return direct_gemm_launch<false>(a, q, mb, nb, nw, st);
}
