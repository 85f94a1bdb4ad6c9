// The LDS-staged tiles (gemm_tile.h) with int8 output on tiled operands.
#include "gemm_tile.h"

void sq_tile_gemm_codes_tiled(const TilePlan& pl, const GemmArgs& a, bool bf16, hipStream_t st)
{
    tile_launch_codes<true>(pl, a, bf16, st);
}
