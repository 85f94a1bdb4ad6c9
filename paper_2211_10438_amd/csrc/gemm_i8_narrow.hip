// INT8 GEMM for few tokens and few output channels (T <= 128 with C_o below 16 per compute unit, T <= 16 up to 1.6 times that), gfx950.
//
// Such a layer is a few megabytes of weights at most and is bound by latency: the time from the first load to the last store,
// not by bandwidth.  (The tile kernels cut C_o into 256-column tiles, 12 workgroups for 3072 columns, each walking its K
// range one barrier after the other, and with a longer K range added a split and a second kernel to sum it.)  Here
//  * a workgroup owns 16 output channels -- one MFMA operand -- and all tokens, so that 3072 channels already make 192
//    workgroups;
//  * its eight waves deal the 64-byte K steps among themselves: no barrier in the K loop, no LDS staging.  In either layout the
//    operands of v_mfma_i32_16x16x64_i8 are 16 rows x 64 bytes as they lie in memory, one 16-byte load per lane, and a wave
//    keeps several steps of loads in flight;
//  * the waves' int32 sums meet in LDS and the dequantizing epilogue of Eq. 2 is applied once: one kernel, no workspace.
// The weights are the first MFMA operand, so that a lane holds four neighbouring output channels of one token.
#include "gemm_args.h"
#include "sqmi_probe.h"

namespace {

constexpr int kNarrowWaves = 8;

// MB: 16-token blocks.  D: K steps of loads in flight per wave.
template <int MB, int D>
__global__ __launch_bounds__(kNarrowWaves * 64, 2) void gemm_i8_narrow_kernel(const GemmArgs p, int tiled, int to_i32, int bf16)
{
    constexpr int NW = kNarrowWaves;
    __shared__ __attribute__((aligned(16))) int red[NW][MB * 16 * 16];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane & 15, chunk = lane >> 4;
    const int n0 = blockIdx.x * 16;
    const int nk = (p.K + 63) >> 6;              // 64-byte K steps
    const int tail = (p.K & 63) >> 4;            // valid 16-byte chunks of the last step (0 = all four)
    // Steps come in pairs, pair wave, wave + NW, ... to this wave: the two halves of a 128-byte line of a row-major operand are
    // then asked for one right after the other by the same wave (an odd last step is followed by itself, its product dropped).
    const int pairs = (nk + 1) >> 1, steps = pairs > wave ? 2 * ((pairs - wave + NW - 1) / NW) : 0;
    auto step_of = [&](int t) { return ((t >> 1) * NW + wave) * 2 + (t & 1); };

    // Rows past the end of an operand re-read its last one (row-major) or lie in the padding of its last block (tiled);
    // their sums are dropped.
    const int64_t kstep = tiled ? 1024 : 64;
    const int in_block = row * 64 + ((chunk ^ ((row >> 1) & 3) ^ ((row >> 3) & 1)) << 4);
    auto base = [&](const int8_t* op, int block, int rows) {
        if (tiled) return op + (int64_t)block * nk * 1024 + in_block;
        const int r = block * 16 + row;
        return op + (int64_t)(r < rows ? r : rows - 1) * p.K + chunk * 16;
    };
    const int8_t* pw = base(p.B, blockIdx.x, p.N);
    const int8_t* pa[MB];
    const int last_block = (p.M - 1) >> 4;
#pragma unroll
    for (int i = 0; i < MB; ++i) pa[i] = base(p.A, i < last_block ? i : last_block, p.M);

    v4i acc[MB];
#pragma unroll
    for (int i = 0; i < MB; ++i) acc[i] = v4i{0, 0, 0, 0};
    if (steps > 0) {
        v4i fw[D], fa[D][MB];
        // step t of this wave (past the end its last one again: the number of loads in flight is the same on every path)
        auto load = [&](int d, int t) {
            int s = step_of(t < steps ? t : steps - 1);
            s = s < nk ? s : nk - 1;
            // chunks past K re-read chunk 0 of the step; the token operand is zeroed there
            const int64_t off = s * kstep - (tail && s == nk - 1 && chunk >= tail ? chunk * 16 : 0);
            fw[d] = __builtin_nontemporal_load((const v4i*)(pw + off));
#pragma unroll
            for (int i = 0; i < MB; ++i) fa[d][i] = *(const v4i*)(pa[i] + off);
        };
#pragma unroll
        for (int d = 0; d < D; ++d) load(d, d);
        for (int t0 = 0; t0 < steps; t0 += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const int t = t0 + d;
                if (t >= steps) break;
                const int s = step_of(t);
                const bool cut = s >= nk || (tail && s == nk - 1 && chunk >= tail);
#pragma unroll
                for (int i = 0; i < MB; ++i) {
                    const v4i a = cut ? v4i{0, 0, 0, 0} : fa[d][i];
                    acc[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fw[d], a, acc[i], 0, 0, 0);
                }
                load(d, t + D);
            }
        }
    }
    // 16x16 accumulator: lane l, register v holds weight row 4 (l >> 4) + v, token l & 15
#pragma unroll
    for (int i = 0; i < MB; ++i) *(v4i*)&red[wave][(i * 16 + row) * 16 + chunk * 4] = acc[i];
    __syncthreads();

    const int tok = threadIdx.x >> 2, col = n0 + (threadIdx.x & 3) * 4;
    if (tok >= MB * 16 || tok >= p.M || col >= p.N) return;
    v4i sum = {0, 0, 0, 0};
#pragma unroll
    for (int w = 0; w < NW; ++w) sum += *(const v4i*)&red[w][threadIdx.x * 4];
    const int64_t o = (int64_t)tok * p.N + col;
    const int ncol = p.N - col < 4 ? p.N - col : 4;
    if (to_i32) {
        if ((p.N & 3) == 0) {
            *(v4i*)(p.acc_out + o) = sum;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (e < ncol) p.acc_out[o + e] = sum[e];
        }
        return;
    }
    const float xs = p.x_scale ? (p.per_token ? p.x_scale[tok] : p.x_scale[0]) : 0.0f;
    const float ws = p.x_scale && !p.w_per_channel ? p.w_scale[0] : 0.0f;
    const uint16_t* R = (const uint16_t*)p.residual;
    uint32_t ob[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int ce = e < ncol ? e : 0;  // (columns past the end: the first one again, not stored)
        const float c = p.x_scale ? xs * (p.w_per_channel ? p.w_scale[col + ce] : ws) : p.alpha;
        const float bias = p.bias ? p.bias[col + ce] : 0.0f;
        const uint32_t rb = R ? (uint32_t)R[o + ce] : 0u;
        ob[e] = bf16 ? dequant_one<true>(sum[e], c, bias, p.bias != nullptr, p.relu != 0, rb, R != nullptr)
                     : dequant_one<false>(sum[e], c, bias, p.bias != nullptr, p.relu != 0, rb, R != nullptr);
    }
    if (p.q8_step) {
        const float delta = p.q8_step[0];
        const float rq = delta > 0.0f ? 1.0f / delta : 0.0f;
        int8_t* dst = code_dst(p.q8_out, tok, col & ~7, p.N, p.q8_tiled != 0) + (col & 7);  // (col & 7 is 0 or 4)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (e < ncol) dst[e] = (int8_t)(bf16 ? requant_code<true>(ob[e], rq) : requant_code<false>(ob[e], rq));
        return;
    }
    uint16_t* dst = (uint16_t*)p.C + o;
    if ((p.N & 3) == 0) {
        *(v2u*)dst = v2u{(ob[0] & 0xffffu) | (ob[1] << 16), (ob[2] & 0xffffu) | (ob[3] << 16)};
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (e < ncol) dst[e] = (uint16_t)ob[e];
    }
}

}  // namespace

// Where it pays, in microseconds: this kernel against the tile and streaming kernels with their K split and reduction, 2100 shapes of
// C_i 64 to 49152, C_o 64 to 6544, 1 to 128 tokens.
//  * Tiled operands (this / others): 16 x 768 -> 3072 4.3 / 6.6, 16 x 5120 -> 3072 7.3 / 11.9, 64 x 5120 -> 768 7.3 / 12.2, 128 x
//    3072 -> 3072 11.4 / 18.7, 16 x 12288 -> 4088 12.7 / 25; but every workgroup reads all tokens, and from some product of tokens
//    and C_i on that decides: 128 x 12288 -> 768 27 / 22, 16 x 49152 -> 768 31 / 20.  That is the fit.  Near one 16-channel unit per
//    compute unit the streaming kernel's split is ahead of it with many tokens and long C_i: 64 x 20480 -> 4088 31.5 / 27.6.
//  * Row-major operands come as sixteen 64-byte pieces per load, and what they cost depends on the row stride: with rows of a
//    multiple of 128 bytes the pieces fall on few channels of the memory.  C_i = 784: 0.5 to 0.8 of the others' time up to 128 tokens and
//    4095 channels (100 x 784 -> 4088 8.1 / 13.7).  C_i = 768 or 896: 32 tokens 7.1 / 6.8, 64 tokens 8.0 / 8.3 and 8.9 / 8.9, 128
//    tokens 10.7 / 12.9 and up to 1.2 times the others' time at 4088 channels.
//  * Between one and 1.6 units per compute unit (tiled, up to 16 tokens) the streaming kernel, one workgroup per compute unit,
//    deals two units to some and leaves the others idle: 20480 -> 5120 31 / 41, 5120 -> 5120 11.4 / 13.1, 16 x 1024 -> 5120 4.8 /
//    5.9 (at 9216 -> 9216, 2.25 units, 24 / 22).  One or two tokens with C_i of 512 to 2048 are the exception, 1 x 1024 -> 5120 6.6 /
//    5.9.
bool sq_narrow_gemm_eligible(int64_t M, int64_t N, int64_t K, int64_t batch, bool tiled)
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

extern "C" int sq_probe_narrow_gemm(int64_t t, int64_t c_i, int64_t c_o, sq_layout layout)
{
    return t > 0 && c_i > 0 && c_o > 0 && sq_narrow_gemm_eligible(t, c_o, c_i, 1, layout == SQ_TILED) ? 1 : 0;
}

void sq_narrow_gemm_launch(const GemmArgs& a, bool to_i32, bool bf16, bool tiled, hipStream_t st)
{
    const dim3 grid((unsigned)((a.N + 15) / 16)), block(kNarrowWaves * 64);
#define SQ_N(MB, D) sq_launch((gemm_i8_narrow_kernel<MB, D>), grid, block, 0, st, a, tiled ? 1 : 0, to_i32 ? 1 : 0, bf16 ? 1 : 0)
    if (a.M <= 16) SQ_N(1, 8);
    else if (a.M <= 32) SQ_N(2, 6);
    else if (a.M <= 64) SQ_N(4, 4);
    else SQ_N(8, 3);
#undef SQ_N
}
