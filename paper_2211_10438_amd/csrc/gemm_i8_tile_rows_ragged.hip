// The LDS-staged tiles (gemm_tile.h) with 16-bit output of rows that are not whole 16-byte pieces, on row-major operands.
#include "gemm_tile.h"

void sq_tile_gemm_ragged_rows(const TilePlan& pl, const GemmArgs& a, bool bf16, int batch, hipStream_t st)
{
    tile_launch_ragged<false>(pl, a, bf16, batch, st);
}
