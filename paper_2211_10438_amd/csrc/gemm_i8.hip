// Host side of the INT8 GEMM: which kernel a layer runs (the direct kernel, the weight-streaming kernels, the LDS-staged tiles of
// gemm_tile.h with or without a K split), the reduction of K splits, and the entry points.
#include <mutex>
#include "gemm_tile_plan.h"
#include "sqmi_probe.h"

namespace {

// Split-K reduction: sums the int32 partial tiles (exact) and applies the same epilogue, four neighbouring columns per
// thread (N % 4 == 0; any other N one column), the partials read 16 bytes at a time, several splits in flight.  One column
// per thread and a 64-bit division per output made it 17-19 us for 512 x 5120 outputs of 4 splits (42 MB).  Short threads: what counts
// is how often each waits for memory, so the scales, bias and residual are under way before the partials are (behind them: 512 x
// 4096 -> 5120 in splits with a residual 33.3 us, now 28.7; 700 x 6000 -> 3000 34.6 / 30.5, the tiles' share of that about 2 us each).
template <bool BF16, int VEC>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const GemmArgs p, int to_i32)
{
    const int64_t total = (int64_t)p.M * p.N;
    const uint32_t per_row = (uint32_t)p.N / VEC;
    const int64_t items = (int64_t)p.M * per_row;
    const uint16_t* R = (const uint16_t*)p.residual;
    float rq = 0.0f;
    if (p.q8_step) {
        const float delta = p.q8_step[0];
        rq = delta > 0.0f ? 1.0f / delta : 0.0f;
    }
    const float xs0 = p.x_scale && !p.per_token ? p.x_scale[0] : 0.0f, ws0 = p.x_scale && !p.w_per_channel ? p.w_scale[0] : 0.0f;
    for (int64_t it = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; it < items; it += (int64_t)gridDim.x * blockDim.x) {
        const int row = (int)(items <= 0xffffffffll ? (uint32_t)it / per_row : it / per_row);
        const int col = (int)(it - (int64_t)row * per_row) * VEC;
        const int64_t idx = it * VEC;
        typedef int vec_t __attribute__((ext_vector_type(VEC)));
        typedef float vecf_t __attribute__((ext_vector_type(VEC)));
        typedef uint16_t vech_t __attribute__((ext_vector_type(VEC)));
        // everything the output needs is asked for before the sums are waited for
        float xs = xs0;
        vecf_t ws, bias;
        vech_t res;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            ws[e] = ws0;
            bias[e] = 0.0f;
            res[e] = 0;
        }
        if (!to_i32) {
            if (p.per_token && p.x_scale) xs = p.x_scale[row];
            if (p.w_per_channel && p.x_scale) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) ws[e] = p.w_scale[col + e];
            }
            if (p.bias) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) bias[e] = p.bias[col + e];
            }
            if (R) res = *(const vech_t*)(R + idx);
        }
        const int32_t* part = p.acc_out + idx;
        vec_t sum = *(const vec_t*)part;
        int s = 1;  // (four at a time without bounds, then what is left at once: with a bound on every load 30 splits take 0.4 us more)
        for (; s + 4 <= p.splits; s += 4) {
            vec_t v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = *(const vec_t*)(part + (s + k) * total);
#pragma unroll
            for (int k = 0; k < 4; ++k) sum += v[k];
        }
        if (s < p.splits) {
            vec_t v[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) v[k] = *(const vec_t*)(part + (s + k < p.splits ? s + k : p.splits - 1) * total);
#pragma unroll
            for (int k = 0; k < 3; ++k)
                if (s + k < p.splits) sum += v[k];
        }
        if (to_i32) {
            *(vec_t*)((int32_t*)p.C + idx) = sum;
            continue;
        }
        uint32_t o[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const float c = p.x_scale ? xs * ws[e] : p.alpha;
            o[e] = dequant_one<BF16>(sum[e], c, bias[e], p.bias != nullptr, p.relu != 0, res[e], R != nullptr) & 0xffffu;
        }
        if (p.q8_step) {
            int8_t* dst = code_dst(p.q8_out, row, col & ~7, p.N, p.q8_tiled != 0) + (col & 7);
#pragma unroll
            for (int e = 0; e < VEC; ++e) dst[e] = (int8_t)requant_code<BF16>(o[e], rq);
        } else {
            uint16_t* dst = (uint16_t*)p.C + idx;
            if constexpr (VEC == 4) {
                *(v2u*)dst = v2u{o[0] | (o[1] << 16), o[2] | (o[3] << 16)};
            } else {
#pragma unroll
                for (int e = 0; e < VEC; ++e) dst[e] = (uint16_t)o[e];
            }
        }
    }
}

// ---------------------------------------------------------------- host side: tile / split choice

constexpr int kNumCU = 256;

// The plan that sizes the workspace (callers keep that size, so its K splits are fixed by the shape), and the plan that runs for up to
// 128 tokens, for short K and for batches; longer layers of more tokens choose their tile below.
TilePlan make_plan(int64_t M, int64_t N, int64_t K, int64_t batch, bool allow_split)
{
    TilePlan pl{};
    pl.bn = 256;
    if (M > 128 && K <= 128) {
        // One or two K steps: the whole range fetched in one go, four small workgroups per CU (see the next case).
        pl.cfg = 8;
        pl.bm = 128;
        pl.bn = 128;
        allow_split = false;
    }
    else if (M > 128 && K <= 256) {
        // Two to four K steps per tile (attention scores, K = head_dim): loading, MFMAs and the epilogue of
        // one tile cannot overlap each other, so several small workgroups share a CU and overlap between
        // themselves; the kernel is bound by writing the output.
        pl.cfg = 7;
        pl.bm = 128;
        pl.bn = 128;
        allow_split = false;
    }
    else if (M > 128) {
        // Compute-bound shapes: time = rounds of tiles over the 256 CUs x cost of one tile; pick the cheapest width.
        // Cost of a tile in microseconds, measured on quantized Gaussian operands (the clock that the power cap allows
        // is part of these figures): K steps x 0.59 + 10 (256x192: fewer MFMAs per operand fragment read), x 0.70 + 18
        // (256x256), x 1.12 + 8 (256x384: 192 accumulator registers per lane, the whole 160 KB of LDS, the epilogue in
        // two halves) with the 32x32x32 MFMA; the 256- and 384-wide tiles also exist with the 16x16x64 MFMA, which
        // draws less power per multiply-accumulate: x 0.66 + 18 and x 1.03 + 8; the 192-wide one too, x 0.52 + 14 (a
        // 5-stage ring: the barrier of a step sits at its start), taken from 192 K steps on.  That form needs an even
        // number of whole K steps and no K split (see the kernel); other shapes keep the 32x32x32 form.
        pl.cfg = 0;
        pl.bm = 256;
        const bool mf16 = (K & 127) == 0;
        const int64_t tm = (M + 255) / 256;
        const int64_t rounds256 = (tm * ((N + 255) / 256) * batch + kNumCU - 1) / kNumCU;
        const int64_t rounds192 = (tm * ((N + 191) / 192) * batch + kNumCU - 1) / kNumCU;
        const int64_t rounds384 = (tm * ((N + 383) / 384) * batch + kNumCU - 1) / kNumCU;
        const double nks = (double)((K + 63) / 64);
        const bool mf16_192 = mf16 && nks >= 192.0;  // (its longer ring costs more per tile: it pays on long K ranges only)
        const double t192 = rounds192 * (mf16_192 ? nks * 0.522 + 14.0 : nks * 0.588 + 10.0);
        const double t256 = rounds256 * (nks * (mf16 ? 0.66 : 0.70) + 18.0);
        const double t384 = rounds384 * (nks * (mf16 ? 1.03 : 1.12) + 8.0);
        double t_now = t256;
        if (t192 < t256) { pl.cfg = 6; pl.bn = 192; t_now = t192; }
        if (t384 < 0.98 * t_now) { pl.cfg = 9; pl.bn = 384; }
    }
    else if (M > 64) { pl.cfg = 1; pl.bm = 128; }
    else if (M > 32) { pl.cfg = 2; pl.bm = 64; }
    else { pl.cfg = 3; pl.bm = 32; }
    pl.tiles_m = (int)((M + pl.bm - 1) / pl.bm);
    pl.tiles_n = (int)((N + pl.bn - 1) / pl.bn);
    const int nk = (int)((K + 63) / 64);
    int splits = 1;
    if (allow_split && batch == 1) {
        const int64_t tiles = (int64_t)pl.tiles_m * pl.tiles_n;
        const int max_splits = nk / 8 > 0 ? nk / 8 : 1;  // at least 8 K steps per split
        if (pl.bm == 256) {
            // Compute-bound tiles: a K split pays (int32 partials through HBM, a second kernel), so it is chosen
            // by a small time model in microseconds: rounds x (K steps x 0.7 + 12 for fill and epilogue), plus,
            // when split, 5 for the reduction launch and the partials written and read back at about 4 TB/s
            // (the write overlaps the GEMM half way).
            double best = 1e30;
            for (int sp = 1; sp <= 8 && sp <= max_splits; ++sp) {
                const int64_t rounds = (tiles * sp + kNumCU - 1) / kNumCU;
                double t_us = (double)rounds * (((nk + sp - 1) / sp) * 0.7 * pl.bn / 256.0 + 12.0);
                if (sp > 1) t_us += 5.0 + 1.5 * sp * (double)M * (double)N * 4.0 / 4e6;
                if (t_us < best * 0.97) { best = t_us; splits = sp; }
            }
        } else if (tiles < 2 * kNumCU) {
            // Weight-streaming shapes: a few workgroups per CU keep every HBM channel busy.
            splits = (int)((2 * kNumCU + tiles - 1) / tiles);
            if (splits > max_splits) splits = max_splits;
            if (splits > 32) splits = 32;
        }
    }
    int per = (nk + splits - 1) / splits;
    splits = (nk + per - 1) / per;  // no empty split
    pl.splits = splits;
    pl.iters_per_split = per;
    if ((K & 127) == 0 && splits == 1) {  // the 16x16x64 form of the tile
        if (pl.cfg == 0) pl.cfg = 10;
        if (pl.cfg == 9) pl.cfg = 11;
        if (pl.cfg == 6 && K >= 192 * 64) pl.cfg = 12;
    }
    return pl;
}

// The tiles of layers with more than 128 tokens and more than 256 input channels.  Microseconds of a K step and of a tile beside its
// steps, row-major and tiled; times = rounds of tiles over the compute units x (steps x step + tile) + the constants below.  Fitted to 1130
// measurements of 91 layers (129 to 4096 tokens, Gaussian codes) when the tiles of pairs of steps had eight waves and all epilogues waited for
// their scales; of the kernels as they are, with weights from memory, the choice costs 2.7 % against the best tile and split of each of 379
// layers that run a tile (121 more than 3 %, 26 more than 10 %, worst 1.31: 1168 x 13184 -> 968 row-major 40.5 us in six splits of 256 x 128, 31.0
// in five of 192 x 160).  All constants fitted anew to 450 such layers came to 2.1 to 2.7 % on 150 others: it is the form of the model that
// does not tell them apart.  It orders tiles; absolute times are corrected in tile_us.  The tiles of pairs of steps (13 to 16) do no better per operation than the wide ones, but leave fewer compute units
// idle (us by graph replay, plan without / with these: 1000 x 9216 -> 9216 row-major 104 / 81, 153 x 3712 -> 30080 45.0 / 33.9, 512 x 20480 -> 5120
// tiled 69 / 61, 2079 x 3328 -> 1352 37.9 / 27.9); the wide ones win from about three rounds on (2048 x 12288 -> 36864 649 / 786), where the
// power cap sets the time: no tile is modelled above the rate measured there.
struct TileCost {
    int cfg, bm, bn;
    bool even;  // needs an even number of whole K steps and no K split
    struct {
        double step, tile;
        double pops;  // what long launches hold (tiled: the power cap), 10^15 operations per second, padding counted
    } us[2];
};
constexpr TileCost kTiles[] = {
    {0, 256, 256, false, {{0.793, 0.9, 2.10}, {0.529, 4.1, 2.45}}},
    {10, 256, 256, true, {{0.655, 3.8, 2.35}, {0.600, 4.0, 2.60}}},
    {6, 256, 192, false, {{0.672, 1.4, 2.00}, {0.515, 2.4, 2.42}}},
    {12, 256, 192, true, {{0.579, 2.6, 2.10}, {0.529, 2.3, 2.66}}},
    {9, 256, 384, false, {{1.266, 4.0, 2.00}, {0.733, 11.2, 2.55}}},
    {11, 256, 384, true, {{1.064, 8.5, 2.35}, {0.836, 8.4, 2.90}}},
    {13, 256, 160, false, {{0.495, 2.0, 2.20}, {0.420, 2.7, 2.50}}},
    {14, 256, 128, false, {{0.429, 1.7, 2.15}, {0.369, 2.5, 2.35}}},
    {15, 192, 224, false, {{0.524, 2.2, 2.15}, {0.454, 2.8, 2.50}}},
    {16, 192, 160, false, {{0.413, 2.1, 2.10}, {0.369, 2.5, 2.30}}},
};

// `sized`: the plan whose K splits the workspace is sized for (not more of them here); kept unless another one is modelled 4 % faster.
// us: modelled time.
TilePlan choose_tile(int64_t M, int64_t N, int64_t K, bool tiled, const TilePlan& sized, double* us)
{
    const int most = sized.splits;
    double sized_us = 1e30;
    const double fixed = tiled ? 2.6 : 2.5, split_us = tiled ? 3.1 : 4.9, part_us = tiled ? 1.97 : 1.78, out_us = tiled ? 0.68 : 0.80;
    const double out = (double)M * (double)N * 1e-6;
    const int nk = (int)((K + 63) / 64);
    TilePlan best{};
    double best_us = 1e30;
    for (const TileCost& c : kTiles) {
        const int64_t tm = (M + c.bm - 1) / c.bm, tn = (N + c.bn - 1) / c.bn;
        const double sustained_us = (double)(tm * tn) * c.bm * c.bn * (double)K * 2e-9 / c.us[tiled].pops;
        for (int sp = 1; sp <= most && (sp == 1 || nk / sp >= 8); ++sp) {
            if (c.even && (sp > 1 || (K & 127))) break;
            const int per = (nk + sp - 1) / sp;
            if ((nk + per - 1) / per != sp) continue;  // (an empty split)
            const int64_t rounds = (tm * tn * sp + kNumCU - 1) / kNumCU;
            double t = (double)rounds * (per * c.us[tiled].step + c.us[tiled].tile) + fixed + (sp > 1 ? split_us + part_us * sp * out : out_us * out);
            if (t < sustained_us) t = sustained_us;
            if (c.cfg == sized.cfg && sp == sized.splits) sized_us = t;
            if (t < best_us) {
                best_us = t;
                best.cfg = c.cfg;
                best.bm = c.bm;
                best.bn = c.bn;
                best.splits = sp;
                best.iters_per_split = per;
                best.tiles_m = (int)tm;
                best.tiles_n = (int)tn;
            }
        }
    }
    if (best_us > 0.96 * sized_us) {
        *us = sized_us;
        return sized;
    }
    *us = best_us;
    return best;
}

// What a call stores: 16-bit or int8 values with scales (a linear layer), 16-bit values with alpha alone, int32 sums.
enum class Epilogue { scales, alpha, sums };

// Time of a tile plan against the direct kernel, fitted to 3500 shapes before the tiles' epilogues stopped waiting for scales (16-bit output, weights in the last-level cache and in memory;
// 4 to 11 % rms).  chosen_us: what choose_tile took the plan for; its model orders tiles of a layer, and leaves out a launch's constant
// part and rows of the output that are not whole 16-byte pieces (odd: they leave element by element).  Without those two 463 x 640 -> 2501
// row-major was taken for 9 us and took 19.
double tile_us(const TilePlan& pl, double M, double N, double K, bool tiled, Epilogue epi, double chosen_us)
{
    const double tiles = (double)((int64_t)pl.tiles_m * pl.tiles_n), out = M * N * 1e-6, w = N * K * 1e-6;
    const double odd = (int64_t)N % (epi == Epilogue::sums ? 4 : 8) ? 1.0 : 0.0, split = pl.splits > 1 ? 1.0 : 0.0, part = pl.splits > 1 ? pl.splits * out : 0.0;
    if (pl.cfg == 8) {
        const double work = tiles / kNumCU * pl.iters_per_split;
        return tiled ? 8.4 + 0.63 * work + 0.155 * out + (1.4 + 1.17 * out) * odd : 8.3 + 0.19 * work + 0.42 * out + (1.6 + 1.12 * out) * odd;
    }
    if (pl.cfg == 7) {
        const double work = tiles / kNumCU * pl.iters_per_split;
        return tiled ? 9.0 + 0.42 * work + (1.4 + 1.10 * out) * odd : 8.9 + 0.56 * out + (1.1 + 0.90 * out) * odd;
    }
    if (pl.bm > 128) return tiled ? 3.3 + 0.90 * chosen_us + (4.0 + 1.2 * out) * odd : 4.0 + 0.875 * chosen_us + (4.2 + 1.5 * out) * odd;
    const double rounds = (double)(((int64_t)tiles * pl.splits + kNumCU - 1) / kNumCU), steps = rounds * pl.iters_per_split;
    switch (pl.bm) {
        case 128:
            return tiled ? 6.0 + 6.9 * rounds + 0.230 * steps + 0.44 * part + 0.266 * w + 2.0 * odd
                         : 11.1 + 1.9 * rounds + 0.300 * steps + 1.97 * part + 0.162 * w + 2.5 * odd;
        case 64:
            return tiled ? 8.0 + 0.6 * rounds + 0.242 * steps + 0.9 * split + 1.71 * part + 0.121 * w + 1.4 * odd
                         : 8.1 + 0.5 * rounds + 0.337 * steps + 0.4 * split + 1.69 * part + 0.224 * w + 1.3 * odd;
        default:
            return tiled ? 6.0 + 0.1 * rounds + 0.223 * steps + 1.9 * split + 2.32 * part + 0.168 * w + 0.2 * odd
                         : 5.6 + 0.6 * rounds + 0.276 * steps + 1.9 * split + 2.90 * part + 0.215 * w + 0.1 * odd;
    }
}

// Sizes of few tokens and few channels, by the shape alone: calls of these sizes ask for no workspace, so they cannot run a K split.  The
// line was drawn where an earlier kernel for them was ahead of the others, and stands because the size of a workspace is part of
// the interface.  The direct kernel takes them all: over 766 such shapes it needs 0.48 of the other path's time, and at most 1.015.
bool few_channels(int64_t M, int64_t N, int64_t K, int64_t batch, bool tiled)
{
    if (batch != 1 || M < 1 || M > 128) return false;
    if (N >= 16 * 256) {
        const int64_t units = (N + 15) / 16;
        return tiled && M <= 16 && units > 256 && units < 410 && !(M <= 2 && K >= 512 && K <= 2048 && units > 264);
    }
    if (!tiled && M > 4) {
        if (K > 1024) return false;
        if (K % 128 != 0) return true;
        return N <= 3072 && !(M > 24 && M <= 32 && K > 640) && !(M > 40 && M <= 64 && K > 768);
    }
    if (tiled && M > 32 && N > 3584 && K > 14336) return false;
    const double per_k = !tiled ? 0.80e-3 : M <= 16 ? 0.62e-3 : M <= 32 ? 0.85e-3 : M <= 64 ? 1.27e-3 : 2.0e-3;
    const double this_us = (tiled ? 3.6 : 5.0) + per_k * (double)K;
    const double others_us = 8.0 + (double)N * (double)K / 3.6e6 + 0.05 * (double)M;
    return this_us < 0.9 * others_us;
}

// Which kernel a call runs.  Apart from the shapes of few tokens and few channels (direct kernel, no further plan) there is always a
// streaming or a tile plan; the direct kernel takes the call where it is modelled to be ahead of it.
struct Path {
    bool stream, tiles;
    int need;  // K splits the workspace is sized for, fixed by the shape
    DirectPlan direct;
};
Path choose(int64_t M, int64_t N, int64_t K, int64_t batch, bool tiled, bool allow_split, Epilogue epi, StreamArgs* sp, TilePlan* pl)
{
    Path p{};
    const bool single = batch == 1;
    const DirectPlan dp = single ? sq_direct_gemm_plan(M, N, K, tiled) : DirectPlan{};
    if (dp.mb && few_channels(M, N, K, batch, tiled)) {
        p.direct = dp;
        return p;
    }
    double us = 0.0;
    if (sq_stream_gemm_plan(M, N, K, batch, tiled, sp) && (sp->gk == 1 || allow_split)) {  // (else the tile kernels)
        p.stream = true;
        p.need = sp->gk;
        us = sp->us;
    } else {
        p.tiles = true;
        *pl = make_plan(M, N, K, batch, allow_split);
        p.need = pl->splits;
        if (single && pl->bm == 256) *pl = choose_tile(M, N, K, tiled, *pl, &us);
        if (single) us = tile_us(*pl, (double)M, (double)N, (double)K, tiled, epi, us);
    }
    // Int32 sums and alpha alone: no scales and biases to wait for at the end of a tile (128 x 128: 8 -> 5 us of fixed time, 256 x 128 2.2 us
    // less; the direct kernel 3.7 -> 3.2).
    if (epi != Epilogue::scales && p.tiles && pl->splits == 1) us -= pl->bm == 32 ? 1.0 : pl->bm == 128 && K > 256 ? 4.5 : 2.2;
    // The margins keep the models' errors from costing where the kernels are close.  Over 4500 shapes the direct kernel was then more than
    // 3 % behind the other in 10 with the weights in the last-level cache and in 49 with them in memory; at 0.95 it would have been 26 and 81.  (Before the
    // tiles' epilogues stopped waiting for scales: of 221 layers of more than 128 tokens it takes now, 12 are more than 3 % behind the tile, the worst
    // 2011 x 512 -> 1088 row-major, 11.3 us against 8.9; it takes 0.705 of their time.)  How
    // long rows of a row-major weight take hangs on more than the model knows (15 x 36336 -> 1360 modelled 25 us, took 38; the tiles 25): of
    // 413 such shapes 1 and 4 are behind, at 0.90 15 and 26.  Few workgroups with long chains are alike (58 x 31152 -> 62: 29 and 39 us, the
    // tiles 15 and 16).
    const double margin = K > 20480 && !tiled && M <= 128 ? 0.80 : p.tiles ? 0.90 : sp->regs ? 0.88 : 0.92;
    const bool chain = K > 12288 && dp.mb && ((M + 16 * dp.mb - 1) / (16 * dp.mb)) * ((N + 16 * dp.nb - 1) / (16 * dp.nb)) < 24;
    if (dp.mb && !chain && dp.us < margin * us) p.direct = dp;
    // Row-major, 33 to 128 tokens: the weights-in-registers kernel where it is modelled clearly ahead of whatever was chosen.  Groups of sizes
    // where it is not ahead for all that, by 1160 shapes (this kernel's time over the other's, weights in the last-level cache / in memory, means):
    //  - rows of whole 128-byte lines, which the direct kernel's small tiles take best: those of 32 x 32 1.23 / 1.06, the others while the
    //    weights fit the L2s of the eight XCDs together 1.22 / 0.95 (82 x 1536 -> 8727 7.7 / 10.1 us cached, 34 x 2432 -> 8320 7.6 / 9.5);
    //  - rows that are not and slabs of at most two units, against the direct kernel 0.97 / 1.02 (116 x 3776 -> 6519 19.2 / 21.2 from memory);
    //  - rows of 8000 and more against the ring's K splits, with slabs of two units 0.90 / 1.06 (63 x 10240 -> 5552 25.0 / 29.3), of three where
    //    whole lines and the four or eight token blocks the ring always has suit that 0.92 / 1.04 (60 x 8192 -> 8240 25.3 / 27.7).
    // The others take 0.73 / 0.85 of the time (400 layers apart from these: one is more than 3 % behind from memory, at 4 %; cached five, the
    // worst but the one above 11 %: 43 x 2752 -> 8448 8.5 / 9.5).
    StreamArgs rows{};
    const int64_t units = (N + 15) / 16, blocks = (M + 15) / 16;
    const bool lines = K % 128 == 0;
    const bool direct_ahead = lines ? (p.direct.mb == 2 && p.direct.nb == 2) || ((p.direct.mb == 1 || p.direct.nb == 2) && N * K <= (int64_t)1 << 25)
                                    : units <= 2 * kNumCU;
    const bool ring_ahead = K >= 8000 && (units <= 2 * kNumCU || (units <= 3 * kNumCU && lines && blocks % 4 == 0));
    const bool other_ahead = p.direct.mb ? direct_ahead : p.stream && ring_ahead;
    if (single && !tiled && !other_ahead && sq_stream_rows_plan(M, N, K, &rows) && rows.us < 0.87 * (p.direct.mb ? dp.us : us) - 1.0) {
        *sp = rows;
        p.stream = true;
        p.tiles = false;
        p.direct = DirectPlan{};
    }
    return p;
}

// allow_split = false: the caller has no workspace to offer (sq_w8a8_bmm), so only plans that finish in one kernel
// are considered.
sq_status run_gemm(GemmArgs a, int64_t batch, bool to_i32, bool bf16, void* workspace, size_t ws_bytes, hipStream_t st,
                   bool tiled = false, bool allow_split = true)
{
    const int64_t total = (int64_t)a.M * a.N;
    auto reduce = [&](void* final_out) {  // a.acc_out = partials [a.splits][M][N]
        a.C = final_out;
        // Four columns per thread from two waves per SIMD of one column each on; below that the longer threads only add latency (us,
        // four / one: 48 x 1024 -> 1024 in two splits 9.2 / 8.6, 64 x 4096 -> 1024 10.4 / 10.2, 130 x 4096 -> 2104 16.5 / 16.8, 512 x
        // 4096 -> 5120 31.1 / 37.2).
        const bool vec = (a.N & 3) == 0 && total >= 131072;
        const int64_t items = vec ? total / 4 : total;
        const unsigned blocks = (unsigned)(items < 256 * 16384 ? (items + 255) / 256 : 16384);
        if (vec && bf16) sq_launch((splitk_reduce_kernel<true, 4>), dim3(blocks), dim3(256), 0, st, a, to_i32 ? 1 : 0);
        else if (vec) sq_launch((splitk_reduce_kernel<false, 4>), dim3(blocks), dim3(256), 0, st, a, to_i32 ? 1 : 0);
        else if (bf16) sq_launch((splitk_reduce_kernel<true, 1>), dim3(blocks), dim3(256), 0, st, a, to_i32 ? 1 : 0);
        else sq_launch((splitk_reduce_kernel<false, 1>), dim3(blocks), dim3(256), 0, st, a, to_i32 ? 1 : 0);
    };
    StreamArgs sp{};
    TilePlan pl{};
    const Path path = choose(a.M, a.N, a.K, batch, tiled, allow_split, to_i32 ? Epilogue::sums : a.x_scale ? Epilogue::scales : Epilogue::alpha, &sp, &pl);
    // (a shape whose workspace is sized for a K split is asked for it also where a kernel that has no use for it takes the call)
    if (path.need > 1 && (!workspace || ws_bytes < (size_t)path.need * total * sizeof(int32_t))) return SQ_ERR_WORKSPACE;
    const int splits = path.stream ? sp.gk : path.tiles ? pl.splits : 1;
    if (path.direct.mb) {
        sq_direct_gemm_launch(a, path.direct.mb, path.direct.nb, path.direct.nw, to_i32, bf16, tiled, st);
        return sq_launch_status();
    }
    if (!path.stream) {
        a.tiles_m = pl.tiles_m;
        a.tiles_n = pl.tiles_n;
        a.iters_per_split = pl.iters_per_split;
    }
    a.splits = splits;
    if (splits > 1) {
        void* final_out = to_i32 ? (void*)a.acc_out : a.C;
        a.acc_out = (int32_t*)workspace;
        if (path.stream) sq_stream_gemm_launch(a, sp, true, false, tiled, st);
        else tile_gemm_launch(pl, a, true, false, 1, st, tiled);
        reduce(final_out);
    } else if (path.stream) {
        sq_stream_gemm_launch(a, sp, to_i32, bf16, tiled, st);
    } else {
        tile_gemm_launch(pl, a, to_i32, bf16, (int)batch, st, tiled);
    }
    return sq_launch_status();
}

bool dims_ok(int64_t t, int64_t c_i, int64_t c_o)
{
    const int64_t lim = (int64_t)1 << 31;
    return t > 0 && c_i > 0 && c_o > 0 && t < lim && c_i < lim && c_o < lim && t * c_o < ((int64_t)1 << 40) &&
           256 * c_i < lim;
}

}  // namespace

extern "C" {

size_t sq_gemm_workspace_bytes(int64_t t, int64_t c_i, int64_t c_o)
{
    if (!dims_ok(t, c_i, c_o)) return 0;
    if (few_channels(t, c_o, c_i, 1, false) && few_channels(t, c_o, c_i, 1, true)) return 0;
    // the layout is not known here: enough for the plan of either
    StreamArgs rows{}, tiles{};
    const int ss_rows = sq_stream_gemm_plan(t, c_o, c_i, 1, false, &rows) ? rows.gk : 0, ss_tiled = sq_stream_gemm_plan(t, c_o, c_i, 1, true, &tiles) ? tiles.gk : 0;
    if (const int ss = ss_rows > ss_tiled ? ss_rows : ss_tiled) return ss > 1 ? (size_t)ss * t * c_o * sizeof(int32_t) : 0;
    TilePlan pl = make_plan(t, c_o, c_i, 1, true);
    return pl.splits > 1 ? (size_t)pl.splits * t * c_o * sizeof(int32_t) : 0;
}

sq_status sq_w8a8_linear(const int8_t* xq, const float* x_scale, int x_scale_per_token, const int8_t* wq,
                         const float* w_scale, int w_scale_per_channel, const float* bias, const void* residual, int relu, void* y,
                         sq_dtype out, int64_t t, int64_t c_i, int64_t c_o, sq_layout layout, void* workspace,
                         size_t ws_bytes, void* stream)
{
    if (!xq || !x_scale || !wq || !w_scale || !y) return SQ_ERR_NULL;
    if (!dims_ok(t, c_i, c_o)) return SQ_ERR_SHAPE;
    if (out != SQ_F16 && out != SQ_BF16) return SQ_ERR_UNSUPPORTED;
    if (layout != SQ_ROW_MAJOR && layout != SQ_TILED) return SQ_ERR_UNSUPPORTED;
    if (layout == SQ_TILED && (c_i & 63)) return SQ_ERR_ALIGN;
    if ((c_i & 15) || !sq_aligned16(xq) || !sq_aligned16(wq) || !sq_aligned16(y) ||
        (residual && !sq_aligned16(residual)) || (workspace && !sq_aligned16(workspace)))
        return SQ_ERR_ALIGN;
    GemmArgs a{};
    a.A = xq; a.B = wq;
    a.M = (int)t; a.N = (int)c_o; a.K = (int)c_i;
    a.lda = c_i; a.ldb = c_i;
    a.C = y; a.x_scale = x_scale; a.per_token = x_scale_per_token ? 1 : 0; a.w_scale = w_scale;
    a.w_per_channel = w_scale_per_channel ? 1 : 0;
    a.bias = bias; a.residual = residual; a.relu = relu ? 1 : 0;
    return run_gemm(a, 1, false, out == SQ_BF16, workspace, ws_bytes, (hipStream_t)stream, layout == SQ_TILED);
}

int sq_probe_narrow_gemm(int64_t t, int64_t c_i, int64_t c_o, sq_layout layout)
{
    return t > 0 && c_i > 0 && c_o > 0 && few_channels(t, c_o, c_i, 1, layout == SQ_TILED) ? 1 : 0;
}

int sq_probe_linear_form(int64_t t, int64_t c_i, int64_t c_o, sq_layout layout)
{
    if (!dims_ok(t, c_i, c_o)) return 0;
    StreamArgs sp{};
    TilePlan pl{};
    const DirectPlan d = choose(t, c_o, c_i, 1, layout == SQ_TILED, true, Epilogue::scales, &sp, &pl).direct;
    return 100 * d.mb + 10 * d.nb + d.nw;
}

int sq_probe_linear_tile(int64_t t, int64_t c_i, int64_t c_o, sq_layout layout)
{
    if (!dims_ok(t, c_i, c_o)) return 0;
    StreamArgs sp{};
    TilePlan pl{};
    const Path p = choose(t, c_o, c_i, 1, layout == SQ_TILED, true, Epilogue::scales, &sp, &pl);
    return p.tiles && !p.direct.mb ? pl.splits * 1000000 + pl.bm * 1000 + pl.bn : 0;
}

sq_status sq_probe_linear_plan(int64_t t, int64_t c_i, int64_t c_o, sq_layout layout, int64_t out[6])
{
    if (!out) return SQ_ERR_NULL;
    if (!dims_ok(t, c_i, c_o)) return SQ_ERR_SHAPE;
    StreamArgs sp{};
    TilePlan pl{};
    const Path p = choose(t, c_o, c_i, 1, layout == SQ_TILED, true, Epilogue::scales, &sp, &pl);
    const int64_t steps = (c_i + 63) / 64;
    const int64_t direct[6] = {0, 100 * p.direct.mb + 10 * p.direct.nb + p.direct.nw, 1, steps, 0, 0};
    const int64_t stream[6] = {1, sp.regs, sp.gk, (int64_t)sp.iters * sp.ksub, sp.gn, sp.units};
    const int64_t tiles[6] = {2, pl.cfg, pl.splits, pl.iters_per_split, pl.tiles_m, pl.tiles_n};
    const int64_t* plan = p.direct.mb ? direct : p.stream ? stream : tiles;
    for (int i = 0; i < 6; ++i) out[i] = plan[i];
    return SQ_OK;
}

// Measurement and test aid: sq_w8a8_linear by the direct kernel with tiles of 16 mb tokens x 16 nb channels.
sq_status sq_probe_linear_blocks(int mb, int nb, int nw, const int8_t* xq, const float* x_scale, int x_scale_per_token, const int8_t* wq,
                                 const float* w_scale, int w_scale_per_channel, const float* bias, const void* residual, int relu,
                                 void* y, sq_dtype out, int64_t t, int64_t c_i, int64_t c_o, sq_layout layout, void* stream)
{
    if (!xq || !x_scale || !wq || !w_scale || !y) return SQ_ERR_NULL;
    if (!dims_ok(t, c_i, c_o)) return SQ_ERR_SHAPE;
    if (out != SQ_F16 && out != SQ_BF16) return SQ_ERR_UNSUPPORTED;
    if (layout != SQ_ROW_MAJOR && layout != SQ_TILED) return SQ_ERR_UNSUPPORTED;
    if (layout == SQ_TILED && (c_i & 63)) return SQ_ERR_ALIGN;
    if ((c_i & 15) || !sq_aligned16(xq) || !sq_aligned16(wq) || !sq_aligned16(y) || (residual && !sq_aligned16(residual))) return SQ_ERR_ALIGN;
    GemmArgs a{};
    a.A = xq; a.B = wq;
    a.M = (int)t; a.N = (int)c_o; a.K = (int)c_i;
    a.lda = c_i; a.ldb = c_i;
    a.C = y; a.x_scale = x_scale; a.per_token = x_scale_per_token ? 1 : 0; a.w_scale = w_scale;
    a.w_per_channel = w_scale_per_channel ? 1 : 0;
    a.bias = bias; a.residual = residual; a.relu = relu ? 1 : 0;
    if (!sq_direct_gemm_launch(a, mb, nb, nw, false, out == SQ_BF16, layout == SQ_TILED, (hipStream_t)stream)) return SQ_ERR_UNSUPPORTED;
    return sq_launch_status();
}

sq_status sq_w8a8_linear_q8(const int8_t* xq, const float* x_scale, int x_scale_per_token, const int8_t* wq,
                            const float* w_scale, int w_scale_per_channel, const float* bias, const void* residual,
                            int relu, sq_dtype mid, const float* y_step, int8_t* yq, sq_layout yq_layout, int64_t t,
                            int64_t c_i, int64_t c_o, sq_layout layout, void* workspace, size_t ws_bytes, void* stream)
{
    if (!xq || !x_scale || !wq || !w_scale || !y_step || !yq) return SQ_ERR_NULL;
    if (!dims_ok(t, c_i, c_o)) return SQ_ERR_SHAPE;
    if (mid != SQ_F16 && mid != SQ_BF16) return SQ_ERR_UNSUPPORTED;
    if (layout != SQ_ROW_MAJOR && layout != SQ_TILED) return SQ_ERR_UNSUPPORTED;
    if (yq_layout != SQ_ROW_MAJOR && yq_layout != SQ_TILED) return SQ_ERR_UNSUPPORTED;
    if (layout == SQ_TILED && (c_i & 63)) return SQ_ERR_ALIGN;
    if (yq_layout == SQ_TILED && (c_o & 63)) return SQ_ERR_ALIGN;
    if ((c_i & 15) || (c_o & 7) || !sq_aligned16(xq) || !sq_aligned16(wq) || !sq_aligned16(yq) ||
        (residual && !sq_aligned16(residual)) || (workspace && !sq_aligned16(workspace)))
        return SQ_ERR_ALIGN;
    GemmArgs a{};
    a.A = xq; a.B = wq;
    a.M = (int)t; a.N = (int)c_o; a.K = (int)c_i;
    a.lda = c_i; a.ldb = c_i;
    a.C = yq;  // never written: the epilogues branch on q8_step
    a.x_scale = x_scale; a.per_token = x_scale_per_token ? 1 : 0; a.w_scale = w_scale;
    a.w_per_channel = w_scale_per_channel ? 1 : 0;
    a.bias = bias; a.residual = residual; a.relu = relu ? 1 : 0;
    a.q8_step = y_step; a.q8_out = yq; a.q8_tiled = yq_layout == SQ_TILED ? 1 : 0;
    return run_gemm(a, 1, false, mid == SQ_BF16, workspace, ws_bytes, (hipStream_t)stream, layout == SQ_TILED);
}

sq_status sq_i8_gemm_i32(const int8_t* xq, const int8_t* wq, int32_t* acc, int64_t t, int64_t c_i, int64_t c_o,
                         sq_layout layout, void* workspace, size_t ws_bytes, void* stream)
{
    if (!xq || !wq || !acc) return SQ_ERR_NULL;
    if (!dims_ok(t, c_i, c_o)) return SQ_ERR_SHAPE;
    if (layout != SQ_ROW_MAJOR && layout != SQ_TILED) return SQ_ERR_UNSUPPORTED;
    if (layout == SQ_TILED && (c_i & 63)) return SQ_ERR_ALIGN;
    if ((c_i & 15) || !sq_aligned16(xq) || !sq_aligned16(wq) || !sq_aligned16(acc) ||
        (workspace && !sq_aligned16(workspace)))
        return SQ_ERR_ALIGN;
    GemmArgs a{};
    a.A = xq; a.B = wq;
    a.M = (int)t; a.N = (int)c_o; a.K = (int)c_i;
    a.lda = c_i; a.ldb = c_i;
    a.acc_out = acc;
    a.C = acc;
    return run_gemm(a, 1, true, false, workspace, ws_bytes, (hipStream_t)stream, layout == SQ_TILED);
}

// ---- sq_w8a8_linear for callers that cannot allocate: the K-split scratch lives in a device array of the library.
// Each GPU the library runs on holds its own copy of the array (at its own address) until the process ends.
}  // extern "C"

namespace {
constexpr size_t kStaticScratchBytes = (size_t)64 << 20;
constexpr int kMaxDevices = 64;
}  // namespace
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
namespace {
std::mutex scratch_mu;
void* scratch_addr[kMaxDevices];  // device address of `scratch` on each device, resolved on first use

// The array's name is a host-side handle only; kernels get the device address hipGetSymbolAddress reports for
// the current device.
sq_status static_scratch(void** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SQ_ERR_HIP;
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (!scratch_addr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return SQ_ERR_HIP;
        scratch_addr[dev] = ptr;
    }
    *out = scratch_addr[dev];
    return SQ_OK;
}
}  // namespace

extern "C" {

size_t sq_static_scratch_bytes(void) { return kStaticScratchBytes; }

sq_status sq_w8a8_linear_noalloc(const int8_t* xq, const float* x_scale, int x_scale_per_token, const int8_t* wq,
                                 const float* w_scale, int w_scale_per_channel, const float* bias, const void* residual,
                                 int relu, void* y, sq_dtype out, int64_t t, int64_t c_i, int64_t c_o, sq_layout layout,
                                 void* stream)
{
    if (!xq || !x_scale || !wq || !w_scale || !y) return SQ_ERR_NULL;
    if (!dims_ok(t, c_i, c_o)) return SQ_ERR_SHAPE;
    const size_t need = sq_gemm_workspace_bytes(t, c_i, c_o);
    if (need > kStaticScratchBytes) return SQ_ERR_WORKSPACE;  // shape beyond the built-in scratch: use sq_w8a8_linear
    void* ws = nullptr;
    if (need) {
        const sq_status st = static_scratch(&ws);
        if (st != SQ_OK) return st;
    }
    // Every K split writes its whole [t, c_o] slice of the partial sums before the reduction reads it, so nothing
    // in the scratch has to start at zero and the previous call's contents do not matter.
    return sq_w8a8_linear(xq, x_scale, x_scale_per_token, wq, w_scale, w_scale_per_channel, bias, residual, relu, y, out,
                          t, c_i, c_o, layout, ws, need ? kStaticScratchBytes : 0, stream);
}

// Attention BMM dispatcher behind sq_w8a8_bmm (arguments already validated).
sq_status sq_internal_bmm(const int8_t* a_, const int8_t* b_, int trans_b, float alpha, void* c, sq_dtype out,
                          int64_t batch, int64_t m, int64_t n, int64_t k, int64_t stride_a, int64_t stride_b,
                          int64_t stride_c, void* stream)
{
    GemmArgs a{};
    a.A = a_; a.B = b_;
    a.M = (int)m; a.N = (int)n; a.K = (int)k;
    a.lda = k;
    a.ldb = trans_b ? k : n;  // trans_b: rows of B are K-contiguous; otherwise B is [k, n]
    a.strideA = stride_a; a.strideB = stride_b; a.strideC = stride_c;
    a.C = c; a.alpha = alpha;
    if (trans_b && sq_strip_bmm_eligible(m, n, k, batch)) {
        sq_strip_bmm_launch(a, (int)batch, out == SQ_BF16, (hipStream_t)stream);
        return sq_launch_status();
    }
    if (!trans_b) {
        sq_pv_bmm_launch(a, (int)batch, out == SQ_BF16, (hipStream_t)stream);
        return sq_launch_status();
    }
    return run_gemm(a, batch, false, out == SQ_BF16, nullptr, 0, (hipStream_t)stream, false, false);
}

}  // extern "C"
