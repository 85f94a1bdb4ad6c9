// The LDS-staged tiles (gemm_tile.h) on row-major operands.
#include "gemm_tile.h"

void sq_tile_gemm_launch_rows(const TilePlan& pl, const GemmArgs& a, bool to_i32, bool bf16, int batch, hipStream_t st)
{
    tile_launch<false>(pl, a, to_i32, bf16, batch, st);
}
