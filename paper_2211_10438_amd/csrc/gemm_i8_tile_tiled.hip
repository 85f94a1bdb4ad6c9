// The LDS-staged tiles (gemm_tile.h) on tiled operands.
#include "gemm_tile.h"

void sq_tile_gemm_launch_tiled(const TilePlan& pl, const GemmArgs& a, bool to_i32, bool bf16, int batch, hipStream_t st)
{
    tile_launch<true>(pl, a, to_i32, bf16, batch, st);
}
