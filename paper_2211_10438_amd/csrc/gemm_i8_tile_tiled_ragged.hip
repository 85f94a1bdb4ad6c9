// The LDS-staged tiles (gemm_tile.h) with 16-bit output of rows that are not whole 16-byte pieces, on tiled operands.
#include "gemm_tile.h"

void sq_tile_gemm_ragged_tiled(const TilePlan& pl, const GemmArgs& a, bool bf16, int batch, hipStream_t st)
{
    tile_launch_ragged<true>(pl, a, bf16, batch, st);
}
