// The LDS-staged tiles (gemm_tile.h) with int8 output on row-major operands.
#include "gemm_tile.h"

void sq_tile_gemm_codes_rows(const TilePlan& pl, const GemmArgs& a, bool bf16, hipStream_t st)
{
    tile_launch_codes<false>(pl, a, bf16, st);
}
