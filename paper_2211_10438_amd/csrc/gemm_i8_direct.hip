// Which tile of the direct kernel (gemm_direct.h) a layer takes, and how long that is expected to last.
#include "gemm_args.h"
#include "sqmi_probe.h"

namespace {

// A time model of each instantiation, microseconds: fixed + per_round x rounds (workgroups over the slots of the chip) + per_wg x
// workgroups of the fullest compute unit + cu x megabytes those pull from their L2 + hbm x megabytes of weights.  Fitted to 590 shapes
// (1 to 2048 tokens, C_i 32 to 65536, C_o 16 to 49152, both layouts, graph replays with rotating weights; about 10 % rms): choosing by it
// costs 2 % against the best instantiation of each shape.  The 10 (tiled) and 12 to 21 (row-major) microseconds per megabyte are 100 and
// 80 to 47 GB/s per compute unit.
struct Cost {
    float fixed, per_round, per_wg, cu, hbm;
};
struct Form {
    int mb, nb, nw;  // tokens / 16, channels / 16, waves
    Cost cost[2];    // row-major, tiled
};
constexpr Form kForms[] = {
    {1, 1, 2, {{3.64f, 0.25f, 0.16f, 14.9f, 0.123f}, {3.19f, 0.57f, 0.09f, 11.0f, 0.095f}}},
    {1, 1, 4, {{3.09f, 0.58f, 0.57f, 12.0f, 0.107f}, {3.46f, 0.00f, 0.45f, 10.8f, 0.093f}}},
    {1, 2, 2, {{3.79f, 0.24f, 0.03f, 14.8f, 0.146f}, {3.36f, 0.15f, 0.22f, 10.3f, 0.107f}}},
    {1, 2, 4, {{3.16f, 0.94f, 0.19f, 13.6f, 0.136f}, {3.18f, 0.38f, 0.52f, 10.3f, 0.099f}}},
    {1, 4, 2, {{4.30f, 0.00f, 0.00f, 16.1f, 0.161f}, {3.58f, 0.34f, 0.37f, 10.5f, 0.110f}}},
    {1, 4, 4, {{3.62f, 0.68f, 0.00f, 14.9f, 0.148f}, {3.06f, 0.92f, 0.72f, 10.1f, 0.105f}}},
    {2, 2, 2, {{3.82f, 0.39f, 0.00f, 14.7f, 0.136f}, {2.92f, 0.83f, 0.34f, 10.0f, 0.094f}}},
    {2, 2, 4, {{2.75f, 0.72f, 0.53f, 11.6f, 0.134f}, {2.75f, 0.67f, 0.79f, 10.0f, 0.089f}}},
    {2, 4, 4, {{4.75f, 0.12f, 0.63f, 21.5f, 0.093f}, {3.06f, 1.02f, 0.88f, 9.8f, 0.103f}}},
    {3, 2, 4, {{3.53f, 0.35f, 0.77f, 13.1f, 0.081f}, {2.78f, 1.19f, 1.07f, 9.7f, 0.072f}}},
    {3, 4, 4, {{4.73f, 0.68f, 0.32f, 21.4f, 0.069f}, {3.20f, 1.13f, 0.79f, 9.6f, 0.087f}}},
    {4, 4, 4, {{4.95f, 1.26f, 0.46f, 22.0f, 0.085f}, {3.04f, 2.00f, 0.74f, 9.5f, 0.096f}}},
    {5, 4, 4, {{5.25f, 1.07f, 0.00f, 21.2f, 0.069f}, {2.72f, 2.78f, 0.39f, 9.6f, 0.083f}}},
    {6, 4, 4, {{5.57f, 1.54f, 0.00f, 21.2f, 0.073f}, {2.87f, 3.59f, 0.26f, 9.9f, 0.067f}}},
    {7, 4, 4, {{6.19f, 1.93f, 0.00f, 21.9f, 0.060f}, {2.78f, 4.28f, 0.29f, 9.6f, 0.081f}}},
};

// Waves per SIMD that the instantiations' registers (tiled) or rings (row-major) allow.
int waves_per_simd(const Form& f, bool tiled) { return tiled && f.nb * f.mb == 1 ? 5 : tiled && f.nb * f.mb == 2 ? 3 : 2; }

}  // namespace

DirectPlan sq_direct_gemm_plan(int64_t M, int64_t N, int64_t K, bool tiled)
{
    constexpr int64_t cus = 256;
    DirectPlan best{};
    for (const Form& f : kForms) {
        const int64_t tm = (M + 16 * f.mb - 1) / (16 * f.mb), wgs = tm * ((N + 16 * f.nb - 1) / (16 * f.nb));
        if (wgs >= ((int64_t)1 << 31) || (f.mb > 1 && 16 * (f.mb - 1) >= M)) continue;  // (a row of 16-token blocks nobody needs)
        const int64_t slots = cus * waves_per_simd(f, tiled) * 4 / f.nw;
        const Cost& c = f.cost[tiled ? 1 : 0];
        const double fullest = (double)((wgs + cus - 1) / cus);
        const double us = c.fixed + c.per_round * (double)((wgs + slots - 1) / slots) + c.per_wg * fullest +
                          c.cu * fullest * (double)(f.mb + f.nb) * (double)K * 15.625e-6 + c.hbm * (double)N * (double)K * 1e-6;
        if (best.mb == 0 || us < best.us) best = DirectPlan{f.mb, f.nb, f.nw, us};
    }
    return best;
}

bool sq_direct_gemm_launch(const GemmArgs& a, int mb, int nb, int nw, bool to_i32, bool bf16, bool tiled, hipStream_t st)
{
    DirectArgs q{};
    q.tiles_m = (a.M + mb * 16 - 1) / (mb * 16);
    q.tiles_n = (a.N + nb * 16 - 1) / (nb * 16);
    q.n_outer = a.N >= a.M ? 1 : 0;
    q.to_i32 = to_i32 ? 1 : 0;
    q.bf16 = bf16 ? 1 : 0;
    return tiled ? sq_direct_gemm_launch_tiled(a, q, mb, nb, nw, st) : sq_direct_gemm_launch_rows(a, q, mb, nb, nw, st);
}
