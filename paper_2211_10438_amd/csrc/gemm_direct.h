// INT8 GEMM whose operands go straight from global memory into MFMA registers, the K range dealt to the waves of a workgroup, gfx950.
//
// For layers with too few output tiles to fill the chip with the LDS-staged tiles (gemm_i8.hip).  Those cut the output into 256-row
// tiles and, where that leaves compute units idle, split K over workgroups, write int32 partial sums to memory and add them in a
// second kernel: a fill, a barrier per K step, a drain and a launch, 18.5 us (now 6.0) for 350 x 1216 -> 1352 whose operands fit one microsecond
// of L2 traffic.  Here
//  * a workgroup owns 16 MB tokens x 16 NB output channels and the whole K range; its two or four waves deal pairs of 64-byte K steps
//    among themselves, each wave with accumulators for the whole tile: no barrier in the K loop, no partial sums in memory;
//  * in the tiled layout the operands of v_mfma_i32_16x16x64_i8 are 1 KB blocks as they lie in memory, one 16-byte load per lane.
//    Row-major operands are dearer: sixteen rows side by side in neighbouring lanes is what the MFMA wants and the address unit takes
//    one lane at a time (64 requests per load against 16 by its counter, 37 against 85 to 130 GB/s per compute unit), so small tiles
//    fetch them through a ring in LDS and the others eight whole lines at a time.  Either way a wave asks for both halves of
//    a 128-byte line in a row: the vector cache fetches whole lines, and a line asked for in two distant steps crosses the L2 twice;
//  * the waves' int32 sums meet in LDS, sixteen 16 x 16 blocks at a time, and the dequantizing epilogue of Eq. 2 is applied once.
// What bounds it: the 64 bytes per clock a compute unit takes from its L2, MB + NB KB per step against MB NB MFMAs, so the largest
// tile that still gives every compute unit work is the best one; for few tokens, the weight stream from HBM.
// The weights are the first MFMA operand, so that a lane holds four neighbouring output channels of one token.
#pragma once
#include "gemm_args.h"

namespace {

// Pairs of K steps in flight per wave: as many as 256 registers per lane hold beside the accumulators.
constexpr int direct_depth(int mb, int nb)
{
    const int d = (212 - mb - nb - 4 * mb * nb) / (8 * (mb + nb));
    return d < 1 ? 1 : d > 4 ? 4 : d;
}

// Row-major operands of small tiles go through a ring of each wave's own in LDS (see there): pairs in it, two waves per SIMD's worth of
// rings in a compute unit; 0: no ring.
constexpr int ring_depth(int mb, int nb)
{
    const int d = (20 << 10) / ((mb + nb) * 2048);
    return d < 2 ? 0 : d > 4 ? 4 : d;
}

template <int MB, int NB, int NW, bool TILED, bool NT>
__global__ __launch_bounds__(NW * 64, 2) void gemm_i8_direct_kernel(const GemmArgs p, const DirectArgs q)
{
    constexpr bool RING = !TILED && ring_depth(MB, NB) > 0;
    constexpr int D = RING ? ring_depth(MB, NB) : direct_depth(MB, NB);
    constexpr int IMAX = 16 / NB;                      // token blocks summed per round: at most 64 KB of LDS
    constexpr int IR = IMAX < MB ? IMAX : MB, AR = IR * NB, ROUNDS = (MB + IR - 1) / IR;
    constexpr int TPP = NW * 16 / NB, QPT = (IR * 16 + TPP - 1) / TPP;  // tokens per pass of the threads, passes per round
    static_assert(NB == 1 || NB == 2 || NB == 4 || NB == 8, "the threads' passes keep their channels");
    constexpr int RED_BYTES = NW * AR * 1024, PAIR = (MB + NB) * 2048, RING_BYTES = RING ? NW * D * PAIR : 0;
    static_assert(RED_BYTES <= 160 * 1024 && RING_BYTES <= 160 * 1024 && (!RING || (D - 1) * (MB + NB) * 2 <= 63), "LDS and vmcnt");
    static_assert(!RING || !NT, "the ring fetches a line by two loads");
    __shared__ __attribute__((aligned(1024))) char smem[RED_BYTES > RING_BYTES ? RED_BYTES : RING_BYTES];
    v4i* const red = (v4i*)smem;  // [NW][AR * 64]
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane & 15, chunk = lane >> 4;

    // Workgroup ids go round-robin to the 8 XCDs: a contiguous range of the tile order each, so that tiles that share operand rows
    // run on one L2.
    int tm, tn;
    {
        const uint32_t xcd = blockIdx.x & 7, j = blockIdx.x >> 3, per = gridDim.x >> 3, r = gridDim.x & 7;
        const uint32_t pid = xcd * per + (xcd < r ? xcd : r) + j;
        const uint32_t inner = (uint32_t)(q.n_outer ? q.tiles_m : q.tiles_n), o = pid / inner, i = pid - o * inner;
        tm = (int)(q.n_outer ? i : o);
        tn = (int)(q.n_outer ? o : i);
    }
    const int m0 = tm * MB * 16, n0 = tn * NB * 16;

    const int nk = (p.K + 63) >> 6;    // 64-byte K steps
    const int pairs = (nk + 1) >> 1, mine = pairs > wave ? (pairs - wave + NW - 1) / NW : 0;  // pairs wave, wave + NW, ...

    // ---- epilogue operands of the thread's output quad: tokens of IR blocks, four neighbouring channels
    const int qd = threadIdx.x % (NB * 4), tk = threadIdx.x / (NB * 4);
    const int col = n0 + qd * 4;
    const int ncol = p.N - col < 4 ? p.N - col : 4;  // (may be negative: no output)
    const bool vec = (p.N & 3) == 0;
    float wsc[4] = {0.0f, 0.0f, 0.0f, 0.0f}, bias[4] = {0.0f, 0.0f, 0.0f, 0.0f}, xs[QPT];
    v2u res[QPT];
    const uint16_t* R = (const uint16_t*)p.residual;
    auto token = [&](int r, int k) { return r * IR * 16 + k * TPP + tk; };  // of the tile; the thread's k-th in round r
    auto has_output = [&](int r, int k) {
        return k * TPP + tk < IR * 16 && token(r, k) < MB * 16 && token(r, k) < p.M - m0 && ncol > 0;
    };
    auto fetch_tokens = [&](int r) {
#pragma unroll
        for (int k = 0; k < QPT; ++k) {
            xs[k] = 0.0f;
            res[k] = v2u{0u, 0u};
            if (q.to_i32 || !has_output(r, k)) continue;
            const int tok = m0 + token(r, k);
            if (p.x_scale) xs[k] = p.per_token ? p.x_scale[tok] : p.x_scale[0];
            if (R) {
                const uint16_t* src = R + (int64_t)tok * p.N + col;
                if (vec) {
                    res[k] = *(const v2u*)src;
                } else {
                    uint32_t v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = src[e < ncol ? e : 0];
                    res[k] = v2u{v[0] | (v[1] << 16), v[2] | (v[3] << 16)};
                }
            }
        }
    };
    // (asked for before the K loop: their latency is then not in front of the first store)
    if (!q.to_i32 && ncol > 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int c = col + (e < ncol ? e : 0);  // (columns past the end: the first one again, not stored)
            if (p.x_scale) wsc[e] = p.w_per_channel ? p.w_scale[c] : p.w_scale[0];
            if (p.bias) bias[e] = p.bias[c];
        }
    }
    fetch_tokens(0);

    // ---- operand addresses: a buffer resource that starts at the tile and ends with the operand, a 32-bit lane offset per 16-row
    // block, the K offset in a scalar.  What lies outside the resource costs no traffic and reads as zero: rows past the end of an
    // operand (their sums are dropped), chunks past K (an offset beyond any resource), and steps past the end of a wave's share (a
    // resource of no bytes), so that the loop has no special last step.
    constexpr int HALF = TILED ? 1024 : 64;  // bytes from one K step to the next
    const int64_t ld16 = TILED ? (int64_t)nk * 1024 : (int64_t)p.K * 16;  // bytes of a 16-row block
    auto left = [&](int first_block, int rows) {  // bytes from a tile's first block to the end of the operand
        const int64_t bytes = TILED ? ((int64_t)((rows + 15) >> 4) - first_block) * ld16 : (int64_t)(rows - first_block * 16) * p.K;
        return (int)(bytes < 0x7fffffff ? bytes : 0x7fffffff);
    };
    int8_t *baseA = const_cast<int8_t*>(p.A) + tm * MB * ld16, *baseB = const_cast<int8_t*>(p.B) + tn * NB * ld16;
    const int lenA = left(tm * MB, p.M), lenB = left(tn * NB, p.N);
    auto swz = [](int r) { return ((r >> 1) & 3) ^ ((r >> 3) & 1); };
    // The row and chunk (of 64 or 128 bytes) of a 16-row block that this lane fetches.  Tiled: its operand chunk.  Ring: four
    // neighbouring lanes the 64 bytes of a row, chunks permuted as in a tiled block.  Else the whole 128-byte lines of eight rows.
    const int load_row = RING ? lane >> 2 : row & 7, load_chunk = RING ? (lane & 3) ^ swz(lane >> 2) : chunk + 4 * (row >> 3);
    const uint32_t v0 = TILED ? (uint32_t)(row * 64 + ((chunk ^ swz(row)) << 4)) : (uint32_t)(load_row * p.K + load_chunk * 16);
    uint32_t vo[MB > NB ? MB : NB];
#pragma unroll
    for (int i = 0; i < (MB > NB ? MB : NB); ++i) vo[i] = v0 + (uint32_t)(i * (int)ld16);

    v4i acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = v4i{0, 0, 0, 0};

    if constexpr (!RING) {
        v4i fa[D][MB][2], fb[D][NB][2];
        // Half h of this wave's pair t: step h of the blocks (tiled), or both steps of rows 8 h .. 8 h + 7 of the blocks (row-major)
        auto load = [&](int d, int t, int h) {
            const int g = wave + t * NW;
            const bool last = g >= pairs - 1, none = g >= pairs || (TILED && h && last && (nk & 1));
            const auto rA = __builtin_amdgcn_make_buffer_rsrc(baseA, 0, none ? 0 : lenA, 0x00027000);
            const auto rB = __builtin_amdgcn_make_buffer_rsrc(baseB, 0, none ? 0 : lenB, 0x00027000);
            uint32_t add = 0;
            if constexpr (!TILED) add = (uint32_t)(h * 8 * p.K) | (last && load_chunk >= (p.K >> 4) - g * 8 ? 0x80000000u : 0u);
            const int off = g * (2 * HALF) + (TILED ? h * HALF : 0);
#pragma unroll
            for (int j = 0; j < NB; ++j) fb[d][j][h] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rB, vo[j] + add, off, NT ? 2 : 0));
#pragma unroll
            for (int i = 0; i < MB; ++i) fa[d][i][h] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rA, vo[i] + add, off, 0));
        };
        // Row-major: lane (r, q) holds chunk q (r < 8) or q + 4 of rows r & 7 and 8 + (r & 7); the operands of the two steps want
        // chunk q and chunk q + 4 of row r.  The lanes 8 apart exchange what the other one needs.
        auto unpack = [&](v4i(&f)[2]) {
            const v4i r0 = f[0], r1 = f[1];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                f[0][e] = __builtin_amdgcn_update_dpp(r0[e], r1[e], 0x128, 0xf, 0xc, false);  // lanes 8-15 of a row: from 8 lanes down
                f[1][e] = __builtin_amdgcn_update_dpp(r1[e], r0[e], 0x128, 0xf, 0x3, false);  // lanes 0-7: from 8 lanes up
            }
        };
        auto multiply = [&](int d, int h) {
            if constexpr (!TILED) {
                if (h == 0) {
#pragma unroll
                    for (int j = 0; j < NB; ++j) unpack(fb[d][j]);
#pragma unroll
                    for (int i = 0; i < MB; ++i) unpack(fa[d][i]);
                }
            }
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[d][j][h], fa[d][i][h], acc[i][j], 0, 0, 0);
        };
        static_for<D>([&](auto d) {
            load(d, d, 0);
            load(d, d, 1);
        });
        for (int t = 0; t < mine; t += D) {
            static_for<D>([&](auto d) {
                // (a refill in front of the use of the old contents would take other registers, and moves: hence the fences.  With
                // one pair of tiled blocks in flight its halves are refilled apart.)
                constexpr bool APART = D == 1 && TILED;
                multiply(d, 0);
                if constexpr (APART) {
                    __builtin_amdgcn_sched_barrier(0);
                    load(d, t + 1, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
                multiply(d, 1);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (!APART) load(d, t + D + d, 0);
                load(d, t + D + d, 1);
                __builtin_amdgcn_sched_barrier(0);
            });
        }
    } else {
        // Row-major operands go through the wave's own ring in LDS (global -> LDS loads, no barrier: nobody else reads it): a register
        // operand wants sixteen rows side by side in neighbouring lanes, and loads so laid out are taken one lane at a time.
        char* const ring = smem + wave * (D * PAIR);
        auto load = [&](int d, int t) {
            const int g = wave + t * NW;
            const bool last = g >= pairs - 1, none = g >= pairs;
            const auto rA = __builtin_amdgcn_make_buffer_rsrc(baseA, 0, none ? 0 : lenA, 0x00027000);
            const auto rB = __builtin_amdgcn_make_buffer_rsrc(baseB, 0, none ? 0 : lenB, 0x00027000);
            const int off = 2 * g * HALF, left = (p.K >> 4) - g * 8;  // chunks from the pair's first to the end of the row
            const uint32_t cut0 = last && load_chunk >= left ? 0x80000000u : 0u, cut1 = last && load_chunk + 4 >= left ? 0x80000000u : 0u;
            char* const dst = ring + d * PAIR;
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                buffer_to_lds<false>(rB, dst + j * 2048, vo[j] | cut0, off);
                buffer_to_lds<false>(rB, dst + j * 2048 + 1024, vo[j] | cut1, off + HALF);
            }
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                buffer_to_lds<false>(rA, dst + (NB + i) * 2048, vo[i] | cut0, off);
                buffer_to_lds<false>(rA, dst + (NB + i) * 2048 + 1024, vo[i] | cut1, off + HALF);
            }
        };
        static_for<D>([&](auto d) { load(d, d); });
        const int frag = row * 64 + ((chunk ^ swz(row)) << 4);
        for (int t = 0; t < mine; t += D) {
            static_for<D>([&](auto d) {
                wait_vmcnt_imm<(D - 1) * (MB + NB) * 2>();  // pair t + d has landed, the younger ones are in flight
                v4i fa[MB][2], fb[NB][2];
                const char* src = ring + d * PAIR + frag;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
#pragma unroll
                    for (int j = 0; j < NB; ++j) fb[j][h] = *(const v4i*)(src + j * 2048 + h * 1024);
#pragma unroll
                    for (int i = 0; i < MB; ++i) fa[i][h] = *(const v4i*)(src + (NB + i) * 2048 + h * 1024);
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // read: the slot may be filled again
                __builtin_amdgcn_sched_barrier(0);
                load(d, t + D + d);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int i = 0; i < MB; ++i)
#pragma unroll
                        for (int j = 0; j < NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[j][h], fa[i][h], acc[i][j], 0, 0, 0);
            });
        }
        wait_vmcnt_imm<0>();  // the loads past the end (of no bytes, but they write LDS) have landed
        __syncthreads();      // everyone is done with its ring: the sums take its place
    }

    float rq = 0.0f;
    if (p.q8_step) {
        const float delta = p.q8_step[0];
        rq = delta > 0.0f ? 1.0f / delta : 0.0f;
    }
    // ---- the waves' sums meet, IR token blocks at a time.  16x16 accumulator: lane l, register v holds channel 4 (l >> 4) + v, token
    // l & 15.  The slots of a channel quad rotate with its number, so that the reads (one token's quads side by side) spread over
    // the banks as the writes do.
    auto slot = [](int blk, int quad, int token) { return blk * 64 + (quad & 3) * 16 + ((token + quad) & 15); };
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        if (r > 0) __syncthreads();  // everyone has read the previous round's sums
#pragma unroll
        for (int i = 0; i < IR; ++i) {
            if (r * IR + i >= MB) continue;
#pragma unroll
            for (int j = 0; j < NB; ++j) red[wave * (AR * 64) + slot(i * NB + j, j * 4 + chunk, row)] = acc[r * IR + i][j];
        }
        if (r > 0) fetch_tokens(r);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < QPT; ++k) {
            if (!has_output(r, k)) continue;
            const int tt = k * TPP + tk, s = slot((tt >> 4) * NB + (qd >> 2), qd, tt & 15);
            v4i sum = red[s];
#pragma unroll
            for (int w = 1; w < NW; ++w) sum += red[w * (AR * 64) + s];
            const int tok = m0 + token(r, k);
            const int64_t o = (int64_t)tok * p.N + col;
            if (q.to_i32) {
                if (vec) {
                    *(v4i*)(p.acc_out + o) = sum;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (e < ncol) p.acc_out[o + e] = sum[e];
                }
                continue;
            }
            uint32_t ob[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float c = p.x_scale ? xs[k] * wsc[e] : p.alpha;
                const uint32_t rb = res[k][e >> 1] >> ((e & 1) * 16);
                ob[e] = q.bf16 ? dequant_one<true>(sum[e], c, bias[e], p.bias != nullptr, p.relu != 0, rb, R != nullptr)
                               : dequant_one<false>(sum[e], c, bias[e], p.bias != nullptr, p.relu != 0, rb, R != nullptr);
            }
            if (p.q8_step) {
                int8_t* dst = code_dst(p.q8_out, tok, col & ~7, p.N, p.q8_tiled != 0) + (col & 7);  // (col & 7 is 0 or 4)
                uint32_t cq[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) cq[e] = (uint32_t)(q.bf16 ? requant_code<true>(ob[e], rq) : requant_code<false>(ob[e], rq));
                if (vec) {
                    *(uint32_t*)dst = pack4_low_bytes(cq[0], cq[1], cq[2], cq[3]);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (e < ncol) dst[e] = (int8_t)cq[e];
                }
                continue;
            }
            uint16_t* dst = (uint16_t*)p.C + o;
            if (vec) {
                *(v2u*)dst = v2u{(ob[0] & 0xffffu) | (ob[1] << 16), (ob[2] & 0xffffu) | (ob[3] << 16)};
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (e < ncol) dst[e] = (uint16_t)ob[e];
            }
        }
    }
}

template <bool TILED> bool direct_gemm_launch(const GemmArgs& a, const DirectArgs& q, int mb, int nb, int nw, hipStream_t st)
{
    const dim3 grid((unsigned)(q.tiles_m * q.tiles_n)), block(nw * 64);
    // The weights' streaming hint where each is read by one workgroup and a load takes whole 128-byte lines: from memory 2 to 20 % faster
    // (tiled; row-major 0 to 5 %).  The ring fetches a line by two loads of 64 bytes, and the hint gives the line up after the
    // first: 16 x 8320 -> 888 took 8.6 us with it, 7.0 without (weights in the last-level cache; from memory 11.3 / 10.8), 16 x 21760 -> 1792
    // 20.4 / 11.9 (23.1 / 22.3), 36 x 14416 -> 17344 118 / 97 (124 / 102).
#define SQ_D(MB, NB, NW)                                                                                           \
    case NW * 256 + MB * 16 + NB: {                                                                                \
        constexpr bool NT = TILED || ring_depth(MB, NB) == 0;                                                      \
        if (NT && q.tiles_m == 1) sq_launch((gemm_i8_direct_kernel<MB, NB, NW, TILED, NT>), grid, block, 0, st, a, q); \
        else sq_launch((gemm_i8_direct_kernel<MB, NB, NW, TILED, false>), grid, block, 0, st, a, q);                \
        return true;                                                                                               \
    }
    switch (nw * 256 + mb * 16 + nb) {
        SQ_D(1, 1, 2) SQ_D(1, 1, 4) SQ_D(1, 2, 2) SQ_D(1, 2, 4) SQ_D(1, 4, 2) SQ_D(1, 4, 4) SQ_D(2, 2, 2) SQ_D(2, 2, 4)
        SQ_D(2, 4, 4) SQ_D(3, 2, 4) SQ_D(3, 4, 4) SQ_D(4, 4, 4) SQ_D(5, 4, 4) SQ_D(6, 4, 4) SQ_D(7, 4, 4)
        default: return false;
    }
#undef SQ_D
}

}  // namespace
