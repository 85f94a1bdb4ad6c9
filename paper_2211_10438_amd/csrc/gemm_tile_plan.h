// Plan of the LDS-staged tile kernels, shared by the host side and the translation units that hold their instantiations.
#pragma once
#include "gemm_args.h"

struct TilePlan {
    int cfg;     // 0: 256x256 (prefill)  1: 128x256  2: 64x256  3: 32x256  6: 256x192
                 // 7: 128x128, three workgroups per CU (short K: the output stream dominates)
                 // 8: 128x128, K <= 128 fetched in one go, four workgroups per CU
                 // 9: 256x384 (a round of tiles saved on wide outputs)
                 // 10, 11, 12: 256x256, 256x384 and 256x192 with the 16x16x64 MFMA
                 // 13, 14, 15, 16: 256x160, 256x128, 192x224 and 192x160 with the 16x16x64 MFMA, K in pairs of steps
    int bm, bn;
    int splits, iters_per_split;
    int tiles_m, tiles_n;
};

// The tiles of a plan: 16-bit values into a.C (ragged: N % 8 != 0), codes into a.q8_out (a.q8_step set; N % 8 == 0), or int32 sums into a.acc_out.
void sq_tile_gemm_launch_rows(const TilePlan& pl, const GemmArgs& a, bool to_i32, bool bf16, int batch, hipStream_t st);
void sq_tile_gemm_launch_tiled(const TilePlan& pl, const GemmArgs& a, bool to_i32, bool bf16, int batch, hipStream_t st);
void sq_tile_gemm_ragged_rows(const TilePlan& pl, const GemmArgs& a, bool bf16, int batch, hipStream_t st);
void sq_tile_gemm_ragged_tiled(const TilePlan& pl, const GemmArgs& a, bool bf16, int batch, hipStream_t st);
void sq_tile_gemm_codes_rows(const TilePlan& pl, const GemmArgs& a, bool bf16, hipStream_t st);
void sq_tile_gemm_codes_tiled(const TilePlan& pl, const GemmArgs& a, bool bf16, hipStream_t st);
static inline void tile_gemm_launch(const TilePlan& pl, const GemmArgs& a, bool to_i32, bool bf16, int batch, hipStream_t st, bool tiled)
{
    if (!to_i32 && a.q8_step) {  // (one batch entry)
        if (tiled) sq_tile_gemm_codes_tiled(pl, a, bf16, st);
        else sq_tile_gemm_codes_rows(pl, a, bf16, st);
    } else if (!to_i32 && (a.N & 7)) {
        if (tiled) sq_tile_gemm_ragged_tiled(pl, a, bf16, batch, st);
        else sq_tile_gemm_ragged_rows(pl, a, bf16, batch, st);
    } else if (tiled) sq_tile_gemm_launch_tiled(pl, a, to_i32, bf16, batch, st);
    else sq_tile_gemm_launch_rows(pl, a, to_i32, bf16, batch, st);
}
