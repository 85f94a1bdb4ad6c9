// Which tile of the direct kernel (gemm_direct.h) a layer takes, and how long that is expected to last.
#include "gemm_args.h"
#include "sqmi_probe.h"

namespace {

// A time model of each instantiation, microseconds: fixed + per_round x rounds (workgroups over the slots of the chip) + per_wg x
// workgroups of the fullest compute unit + cu x megabytes those pull from their L2 + hbm x megabytes of weights.  Fitted to 4500 shapes
// (1 to 4096 tokens, C_i 16 to 50000, C_o 16 to 40000, both layouts), each the geometric mean of a replay with the weights in
// the last-level cache and one with them in memory (5 to 11 % rms): choosing by it costs 0.5 % against the best instantiation of each shape
// (row-major 1 %).  One shape in six has K <= 256: without them the fixed work of a workgroup, its sums and stores, went
// into the other terms, and 1000 x 64 -> 14900 row-major was modelled at 8 us and took 55.  The 11 (tiled) and 11 to 22 (row-major)
// microseconds per megabyte are 90 and 90 to 45 GB/s per compute unit.
struct Cost {
    float fixed, per_round, per_wg, cu, hbm;
};
struct Form {
    int mb, nb, nw;  // tokens / 16, channels / 16, waves
    Cost cost[2];    // row-major, tiled
};
constexpr Form kForms[] = {
    {1, 1, 2, {{2.49f, 1.15f, 0.31f, 16.9f, 0.066f}, {3.33f, 0.00f, 0.35f, 14.3f, 0.056f}}},
    {1, 1, 4, {{2.84f, 0.36f, 0.93f, 11.4f, 0.097f}, {3.25f, 0.00f, 0.65f, 13.1f, 0.077f}}},
    {1, 2, 2, {{2.69f, 0.96f, 0.35f, 15.3f, 0.106f}, {3.22f, 0.12f, 0.50f, 12.3f, 0.080f}}},
    {1, 2, 4, {{2.76f, 0.61f, 0.85f, 12.7f, 0.117f}, {3.30f, 0.00f, 0.91f, 12.2f, 0.081f}}},
    {1, 4, 2, {{2.71f, 1.13f, 0.47f, 14.8f, 0.123f}, {3.02f, 0.55f, 0.88f, 11.5f, 0.090f}}},
    {1, 4, 4, {{2.56f, 0.86f, 0.93f, 12.0f, 0.141f}, {2.89f, 0.45f, 1.49f, 11.3f, 0.095f}}},
    {2, 2, 2, {{2.71f, 1.54f, 0.28f, 14.6f, 0.111f}, {3.45f, 0.51f, 0.62f, 11.4f, 0.077f}}},
    {2, 2, 4, {{2.73f, 0.85f, 0.75f, 12.8f, 0.119f}, {3.39f, 0.00f, 1.22f, 11.4f, 0.091f}}},
    {2, 4, 4, {{2.56f, 2.53f, 0.51f, 21.2f, 0.094f}, {2.95f, 1.20f, 1.23f, 11.3f, 0.091f}}},
    {3, 2, 4, {{3.06f, 1.10f, 0.87f, 12.8f, 0.097f}, {3.18f, 0.85f, 1.45f, 10.9f, 0.079f}}},
    {3, 4, 4, {{2.56f, 2.95f, 0.46f, 21.3f, 0.068f}, {2.83f, 1.81f, 0.98f, 11.0f, 0.088f}}},
    {4, 4, 4, {{2.95f, 3.09f, 1.13f, 21.7f, 0.099f}, {2.89f, 2.22f, 1.22f, 11.0f, 0.081f}}},
    {5, 4, 4, {{2.45f, 4.00f, 0.36f, 20.1f, 0.082f}, {2.49f, 3.15f, 0.74f, 11.1f, 0.075f}}},
    {6, 4, 4, {{2.72f, 4.34f, 0.56f, 20.6f, 0.063f}, {2.85f, 3.36f, 1.01f, 11.2f, 0.054f}}},
    {7, 4, 4, {{2.85f, 4.89f, 0.63f, 20.9f, 0.086f}, {2.99f, 3.73f, 1.23f, 10.7f, 0.079f}}},
};

// Waves per SIMD that the instantiations' registers (tiled) or rings (row-major) allow.
int waves_per_simd(const Form& f, bool tiled) { return tiled && f.nb * f.mb == 1 ? 5 : tiled && f.nb * f.mb == 2 ? 3 : 2; }

// Workgroups of a launch, 0 where it has to go to another kernel: HIP cuts a launch of 2^32 threads or more without an error, and the kernel
// counts tokens and channels in 32 bits, those between the end of an operand and the end of its last tile included.
int64_t workgroups(int64_t M, int64_t N, int mb, int nb, int nw)
{
    constexpr int64_t last = ((int64_t)1 << 31) - 128;  // (the largest tile has 112 tokens)
    if (M > last || N > last) return 0;
    const int64_t wgs = ((M + 16 * mb - 1) / (16 * mb)) * ((N + 16 * nb - 1) / (16 * nb));
    return wgs * nw * 64 < ((int64_t)1 << 32) ? wgs : 0;
}

}  // namespace

DirectPlan sq_direct_gemm_plan(int64_t M, int64_t N, int64_t K, bool tiled)
{
    constexpr int64_t cus = 256;
    DirectPlan best{};
    for (const Form& f : kForms) {
        const int64_t wgs = workgroups(M, N, f.mb, f.nb, f.nw);
        if (!wgs || (f.mb > 1 && 16 * (f.mb - 1) >= M)) continue;  // (a row of 16-token blocks nobody needs)
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
    if (!workgroups(a.M, a.N, mb, nb, nw)) return false;
    DirectArgs q{};
    q.tiles_m = (a.M + mb * 16 - 1) / (mb * 16);
    q.tiles_n = (a.N + nb * 16 - 1) / (nb * 16);
    q.n_outer = a.N >= a.M ? 1 : 0;
    q.to_i32 = to_i32 ? 1 : 0;
    q.bf16 = bf16 ? 1 : 0;
    return tiled ? sq_direct_gemm_launch_tiled(a, q, mb, nb, nw, st) : sq_direct_gemm_launch_rows(a, q, mb, nb, nw, st);
}
