// INT8 x INT8 -> INT32 MFMA GEMM / batched GEMM for gfx950 with a fused dequantizing epilogue.
//
// Computes the integer contraction of Eq. 2, acc[m, n] = sum_k A[m, k] * B[n, k] (both operands
// K-contiguous: activations [T, C_i], prepared weights [C_o, C_i]), and applies the outer-dimension
// scaling of Eq. 2 (per-token Delta_X times Delta_W, optional bias / ReLU / residual) to the int32
// accumulators while they are still in registers.
//
// Design (CDNA4):
//  * Three K loops: v_mfma_i32_32x32x32_i8 with one 64-byte K step per stage (any K, K splits, batches), v_mfma_i32_16x16x64_i8
//    the same way (MF = 16: an even number of whole steps, no split), and v_mfma_i32_16x16x64_i8 with pairs of steps per stage (PAIR).
//  * One wave owns a (MI*MF) x (NI*MF) block of accumulators; the tiles of 192 and 256 rows run 8 waves = 2 per SIMD, so one
//    wave's barrier / LDS waits are covered by the other wave's MFMAs (PAIR: 4 waves, which cover their own).
//  * Operand tiles travel HBM -> LDS with global_load_lds_dwordx4 (PAIR: buffer loads, whose bounds stand in for clamps; no VGPR
//    staging), NSTAGE deep.
//    LDS holds a tile as 16-row blocks of 1 KB, row-major (64 B per row) with the four 16-byte
//    K-chunks of a row XOR-permuted: (a) one wave-wide load instruction fills a block from 16 rows
//    x 64 contiguous bytes of global memory, four neighbouring lanes per row (coalesced), and (b)
//    the ds_read_b128 operand reads of the MFMAs spread over all banks.
//  * One s_barrier per 64-wide K step (PAIR: one per pair of steps); operand fragments are
//    double buffered in registers, so that the LDS reads of the next part of a step are in flight while this part's MFMAs issue.
//  * Tiles are enumerated XCD-aware: the workgroups an XCD runs concurrently cover a compact
//    block of output tiles, so its L2 serves the shared A rows / B rows.
//  * Optional split-K writes int32 partial tiles to a workspace, reduced (exactly, int32) by a
//    second small kernel that also runs the epilogue.
#pragma once
#include <type_traits>

#include "gemm_tile_plan.h"

namespace {

// What a tile stores: 16-bit values in whole 16-byte pieces, the same where rows are not whole pieces, int8 codes, int32 sums.  Each has kernels of its
// own: as branches of one kernel the rarer stores cost the first some 0.2 to 0.5 us a launch (scalar registers, kernel arguments loaded late, residual
// pieces fetched branch by branch), e.g. 300 x 4096 -> 16384 tiled 28.4 / 28.9, 991 x 864 -> 3624 row-major with a residual 14.0 / 14.7.
enum { EPI_DEQUANT = 0, EPI_I32 = 1, EPI_CODES = 2, EPI_RAGGED = 3 };

// BM x BN output tile per workgroup, WGM x WGN waves, BK = 64 bytes of K per pipeline stage.
// B is [N, K] (K-contiguous rows, like A).
//
// LAY selects the operand layouts in global memory:
//   LAY_ROWS  A [M, K] and B [N, K] row-major (K contiguous);
//   LAY_TILED A and B in the tiled layout of sq_layout SQ_TILED: 16-row x 64-byte blocks of 1 KB,
//             stored block-row-major, each block an exact image of the LDS block (chunk permutation
//             included).  One wave-wide load then copies 1 KB of contiguous global memory -- eight whole
//             128-byte lines instead of sixteen 64-byte row segments -- which is what the L2 -> CU path
//             serves best.
enum { LAY_ROWS = 0, LAY_TILED = 2 };

//
// ONESHOT (host guarantees K <= 64 * (NSTAGE - 1)): the whole K range is fetched up front into NSTAGE - 1
// buffers, no refills, no barriers in the K loop.  Used for attention scores (K = head_dim), where the
// kernel is bound by writing its output and several small workgroups per CU (OCC) overlap each other's
// load, MFMA and store phases.
//
// MF selects the MFMA shape: 32 = v_mfma_i32_32x32x32_i8 (two per 64-byte K step and accumulator block), 16 =
// v_mfma_i32_16x16x64_i8 (one per K step; a 1 KB LDS block is exactly one operand).  On quantized operands the matrix
// pipes draw less power per multiply-accumulate in the 16x16x64 shape (a register-fed loop of it sustains 4.1-4.2 POP/s
// under the socket's power cap where the 32x32x32 shape sustains 3.6), and the compute-bound tiles run at that cap.
//
// PAIR (with MF = 16, single launches): a stage is a pair of K steps, 128 bytes of every row, and the ring three stages.  A wave asks
// for both halves of a row's 128-byte line one right after the other, so that a row-major operand's lines cross the L2 once (by counter
// the 256 x 192 tile with 64-byte steps asks the L2 for 12.8 million lines where the tiled layout needs 6.2).  Any number of steps, K
// tails and K splits: what is not there is outside the buffers and arrives as zeros.
template <int BM, int BN, int WGM, int WGN, int NSTAGE, int EPI, bool BF16, int LAY, int OCC = 1, bool ONESHOT = false, int MF = 32, bool PAIR = false>
__global__ __launch_bounds__(WGM* WGN * 64, OCC) void gemm_i8_kernel(const GemmArgs p)
{
    constexpr bool TILED = LAY == LAY_TILED;
    constexpr int NW = WGM * WGN, BK = 64;
    constexpr int WM = BM / WGM, WN = BN / WGN, MI = WM / MF, NI = WN / MF;
    constexpr int AV = MF * MF / 64;  // accumulator registers per block
    constexpr int QG = AV / 4;        // runs of four neighbouring output columns a lane holds per block
    static_assert(MF == 32 || (MF == 16 && !ONESHOT && (PAIR ? NW == 4 && MI >= 6 && MI <= 8 && NI >= 4 : MI == 4 && NI % 2 == 0 && NI >= 6)), "MFMA shape");
    static_assert(!PAIR || (MF == 16 && NSTAGE == 3), "pairs of steps");
    constexpr int A_BYTES = BM * BK, B_BYTES = BN * BK, STAGE = (A_BYTES + B_BYTES) * (PAIR ? 2 : 1);
    constexpr int RBA = BM / 16, RBB = BN / 16;  // 16-row blocks per operand tile
    constexpr int SA = (RBA + NW - 1) / NW, SB = (RBB + NW - 1) / NW;
    constexpr int LPS = SA + SB;          // vector-memory loads per wave per stage
    static_assert(WM % MF == 0 && WN % MF == 0, "wave tile must be a multiple of the MFMA block");
    static_assert(NSTAGE >= 3 && (NSTAGE - 2) * LPS <= 63, "pipeline depth exceeds the 6-bit vmcnt");
    static_assert(NSTAGE * STAGE <= 160 * 1024, "LDS budget");
    // The epilogue stages the 16-bit tile in LDS; a tile too large for that goes in EG groups of GR rows.
    constexpr int EG = BM * (BN * 2 + 16) <= 160 * 1024 ? 1 : 2;
    constexpr int GR = BM / EG;
    constexpr int EPI_VEC = GR * (BN * 2 + 16);  // behind it the scales and biases of the tile's columns and the scales of its rows
    constexpr int EPI_BYTES = EPI != EPI_I32 ? EPI_VEC + (2 * BN + BM) * 4 : 0;
    static_assert(BN <= NW * 64 && BM <= NW * 64, "a thread fetches one column's and one row's");
    constexpr int RING_BYTES = (ONESHOT ? NSTAGE - 1 : NSTAGE) * STAGE;
    constexpr int SMEM_BYTES = RING_BYTES > EPI_BYTES ? RING_BYTES : EPI_BYTES;
    static_assert(SMEM_BYTES <= 160 * 1024, "LDS budget");
    __shared__ __attribute__((aligned(1024))) char smem[SMEM_BYTES];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave / WGN, wn = wave % WGN;

    // ---- which tile: hardware deals consecutive workgroup ids round-robin to the 8 XCDs; give
    // each XCD a contiguous range of the logical order, and make that order walk groups of 8
    // m-tiles column by column so that concurrently running tiles share operand rows in L2.
    // Batched launches (attention heads) are enumerated the same way over (batch, tile) jointly: an XCD
    // then works through whole heads, and the tiles of a head that share its Q / K / V rows run together.
    const int64_t total = (int64_t)gridDim.x * gridDim.y;
    int64_t pid;
    {
        const int64_t wg = (int64_t)blockIdx.y * gridDim.x + blockIdx.x, j = wg >> 3;
        const int xcd = (int)(wg & 7);
        const int64_t q = total >> 3;
        const int r = (int)(total & 7);
        pid = xcd * q + (xcd < r ? xcd : r) + j;
    }
    const int tiles = p.tiles_m * p.tiles_n;
    const int per_batch = (int)gridDim.x;  // tiles * splits
    const int batch = (int)(pid / per_batch);
    const int pin = (int)(pid - (int64_t)batch * per_batch);
    const int split = pin / tiles;
    int tm, tn;
    {
        const int t = pin - split * tiles;
        constexpr int GM = 8;
        const int per_group = GM * p.tiles_n;
        const int g = t / per_group, first_m = g * GM;
        const int gsz = (p.tiles_m - first_m) < GM ? (p.tiles_m - first_m) : GM;
        const int in = t - g * per_group;
        tm = first_m + in % gsz;
        tn = in / gsz;
    }
    const int m0 = tm * BM, n0 = tn * BN;
    const int nk_total = (p.K + BK - 1) / BK;
    const int kbeg = split * p.iters_per_split;
    const int nk = (nk_total - kbeg) < p.iters_per_split ? (nk_total - kbeg) : p.iters_per_split;
    const int tail_chunks = (p.K & (BK - 1)) >> 4;  // valid 16-byte chunks of the last K step (0 = all 4)

    // Tiled operands: a 16-row block row is 16*K contiguous bytes and a K step advances 1 KB.
    constexpr int KSTEP = TILED ? 1024 : BK;
    const int8_t* Ab = p.A + (int64_t)batch * p.strideA + (int64_t)m0 * p.lda + (int64_t)kbeg * KSTEP;
    const int8_t* Bb = p.B + (int64_t)batch * p.strideB + (int64_t)n0 * p.ldb + (int64_t)kbeg * KSTEP;

    // ---- global -> LDS load slots of this wave.  Slot i moves 16-row block (i*NW + wave), 1 KB per
    // stage.  Lane l lands at LDS byte l*16 of the block, i.e. the block is row-major (64 B per row),
    // and fetches row (l >> 2): four neighbouring lanes read one contiguous 64-byte segment, which
    // the vector memory path coalesces.  Inside a row the four 16-byte chunks are permuted
    // (position = chunk ^ swz(row)) so that the MFMA operand reads below stay bank-conflict free.
    auto swz = [](int r) { return ((r >> 1) & 3) ^ ((r >> 3) & 1); };
    const int chunk = (lane & 3) ^ swz(lane >> 2);
    uint32_t offA[SA], offB[SB];
    int ldsA[SA], ldsB[SB];
#pragma unroll
    for (int i = 0; i < SA; ++i) {
        const int rb = (i * NW + wave) % RBA;  // wraps only when RBA is not a multiple of NW: a benign duplicate
        if constexpr (TILED) {
            const int last_rb = (p.M - 1 - m0) >> 4;  // ragged M: re-read the last valid block row
            offA[i] = (uint32_t)((rb < last_rb ? rb : last_rb) * 16 * (int)p.lda + lane * 16);
        } else {
            int row = rb * 16 + (lane >> 2);
            const int last = p.M - 1 - m0;
            row = row < last ? row : last;
            offA[i] = (uint32_t)(row * (int)p.lda + chunk * 16);
        }
        ldsA[i] = rb * 1024;
    }
#pragma unroll
    for (int i = 0; i < SB; ++i) {
        const int rb = (i * NW + wave) % RBB;
        if constexpr (TILED) {
            const int last_rb = (p.N - 1 - n0) >> 4;
            offB[i] = (uint32_t)((rb < last_rb ? rb : last_rb) * 16 * (int)p.ldb + lane * 16);
        } else {
            int row = rb * 16 + (lane >> 2);
            const int last = p.N - 1 - n0;
            row = row < last ? row : last;
            offB[i] = (uint32_t)(row * (int)p.ldb + chunk * 16);
        }
        ldsB[i] = A_BYTES + rb * 1024;
    }

    // K tail (K % 64 != 0 happens only in the globally last K step): lanes whose chunk lies beyond K
    // re-read chunk 0 (valid memory); their A fragments are zeroed in registers before the MFMAs.
    const bool has_tail = tail_chunks != 0 && (kbeg + nk == nk_total);
    auto issue_stage = [&](int kt, int buf) {
        const int8_t* a = Ab + (int64_t)kt * KSTEP;
        const int8_t* b = Bb + (int64_t)kt * KSTEP;
        char* base = smem + buf * STAGE;
        const uint32_t back = (has_tail && kt == nk - 1 && chunk >= tail_chunks) ? (uint32_t)chunk * 16u : 0u;
#pragma unroll
        for (int i = 0; i < SA; ++i)
            __builtin_amdgcn_global_load_lds(GPTR(a + (offA[i] - back)), LPTR(base + ldsA[i]), 16, 0, 0);
#pragma unroll
        for (int i = 0; i < SB; ++i)
            __builtin_amdgcn_global_load_lds(GPTR(b + (offB[i] - back)), LPTR(base + ldsB[i]), 16, 0, 0);
    };

    // ---- MFMA operand fragments.  For the 32x32x32 MFMA lane l feeds row (l & 31) with the 16
    // bytes of K-chunk kk*2 + (l >> 5) of the 64-wide K step; chunk c of row r sits at position
    // c ^ swz(r), and kk only flips bit 1 of the position: byte address ^ 32.
    // For the 16x16x64 MFMA lane l feeds row (l & 15) with the 16 bytes of K-chunk (l >> 4): one 1 KB block, whole.
    const int frow = lane & 15;
    const int lane_off = MF == 32 ? ((lane & 31) >> 4) * 1024 + frow * 64 + (((lane >> 5) ^ swz(frow)) * 16)
                                  : frow * 64 + (((lane >> 4) ^ swz(frow)) * 16);
    constexpr int FB = PAIR ? 2048 : 1024;  // bytes from one 16-row block of a stage to the next
    const int fragA0 = wm * (WM / 16) * FB + lane_off;
    const int fragB0 = RBA * FB + wn * (WN / 16) * FB + lane_off;

    // ---- what the epilogue needs beside the sums: per column scale and bias, per row scale, one of each for a thread to fetch, and the
    // tile of the residual, 16 bytes of a row at a time.  PRE: on their way during the K loop (the tiles of pairs of steps have the registers);
    // fetched behind it they cost 3 us a launch.  1000 x 256 -> 9216, us, before / now: 12.2 / 9.6, with a residual and a step per channel
    // 18.3 / 11.5; 1000 x 9216 -> 9216 with both 90.6 / 86.5 (the power cap takes the rest back).
    constexpr bool PRE = EPI != EPI_I32 && PAIR, PRE_RES = PRE && EPI != EPI_RAGGED;
    constexpr int CPR = BN / 8;                             // 16-byte pieces per tile row
    constexpr int RCH = (GR * CPR + NW * 64 - 1) / (NW * 64);  // of them per thread
    const uint16_t* R = (const uint16_t*)p.residual;
    constexpr bool WHOLE = EPI != EPI_RAGGED;               // N % 8 == 0: 16-byte pieces never straddle the row end and stay aligned
    float col_scale = 0.0f, col_bias = 0.0f, row_scale = 0.0f;
    constexpr bool FULL = MI * NI * AV >= 192;              // the sums leave few registers: one piece more in flight and they spill
    constexpr int RG = PRE || RCH <= 4 ? RCH : FULL ? 2 : 4;  // ... in flight at a time
    v4u rpre[RG];
    auto fetch_scales = [&]() {
        const int t = (int)threadIdx.x, col = n0 + t, row = m0 + t;
        if (t < BN && col < p.N) {
            col_scale = !p.x_scale ? p.alpha : p.w_per_channel ? p.w_scale[col] : p.w_scale[0];
            if (p.bias) col_bias = p.bias[col];
        }
        if (t < BM && row < p.M) row_scale = !p.x_scale ? 1.0f : p.per_token ? p.x_scale[row] : p.x_scale[0];
    };
    auto fetch_residual = [&](int g0, int k0) {
#pragma unroll
        for (int k = 0; k < RG; ++k) {
            const int q = (int)threadIdx.x + (k0 + k) * NW * 64, r = q / CPR, row = m0 + g0 + r, col = n0 + (q - r * CPR) * 8;
            if (q < GR * CPR && row < p.M && col < p.N) rpre[k] = *(const v4u*)(R + (int64_t)row * p.N + col);
        }
    };
    if constexpr (PRE) fetch_scales();

    typedef int acc_t __attribute__((ext_vector_type(AV)));
    acc_t acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int v = 0; v < AV; ++v) acc[i][j][v] = 0;

    if constexpr (MF == 32) {
    v4i fa0[MI], fb0[NI], fa1[MI], fb1[NI];

    auto read_frags = [&](v4i(&fa)[MI], v4i(&fb)[NI], int buf, int kk) {
        const char* sa = smem + buf * STAGE + (fragA0 ^ (kk * 32));
        const char* sb = smem + buf * STAGE + (fragB0 ^ (kk * 32));
#pragma unroll
        for (int i = 0; i < MI; ++i) fa[i] = *(const v4i*)(sa + i * 2048);
#pragma unroll
        for (int j = 0; j < NI; ++j) fb[j] = *(const v4i*)(sb + j * 2048);
    };
    auto mfma_all = [&](const v4i(&fa)[MI], const v4i(&fb)[NI]) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fb[j], fa[i], acc[i][j], 0, 0, 0);
    };
    // (B rows feed the MFMA's first operand: each accumulator block is the transpose of its 32x32 output
    // block, so a lane ends up with runs of four neighbouring output columns of one row -- see the epilogue.)
    // Scheduling hint for one half step (MI+NI fragment reads of the next half, MI*NI MFMAs of this
    // one): interleave the LDS reads with the MFMAs so the four waves of the workgroup do not hit
    // the LDS pipe in one burst.
    auto interleave_hint = [&](auto NV) {
        // one MFMA, one DS read (and, in the half step that refills a buffer, one global->LDS load)
        // per group; the MFMAs left over close the half step, which gives the last read time to land
        // before the next half step waits for it.
        constexpr int READS = MI + NI, MFMAS = MI * NI, VMEM = decltype(NV)::value;
        constexpr int GROUPS = READS > VMEM ? READS : VMEM;
#pragma unroll
        for (int r = 0; r < GROUPS; ++r) {
            if (r < MFMAS) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if (r < VMEM) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            if (r < READS) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        if (MFMAS > GROUPS) __builtin_amdgcn_sched_group_barrier(0x008, MFMAS - GROUPS, 0);
    };

    // ---- pipeline prologue: stages 0 .. NSTAGE-2 in flight, stage 0 landed, first fragments read.
    // Every K step issues exactly one stage of loads; past the end of the K range the last stage is
    // simply fetched again into a buffer nobody reads.  That keeps the number of loads in flight
    // constant (one immediate s_waitcnt value) and the loop body free of branches, so the loads and
    // LDS reads can be interleaved with the MFMAs by the scheduler hints below.
#pragma unroll
    for (int s = 0; s < NSTAGE - 1; ++s) {
        if constexpr (ONESHOT) {
            if (s < nk) issue_stage(s, s);
        } else {
            issue_stage(s < nk ? s : nk - 1, s);
        }
    }
    if constexpr (ONESHOT) {
        wait_vmcnt_imm<0>();
    } else {
        wait_vmcnt_imm<(NSTAGE - 2) * LPS>();
    }
    __builtin_amdgcn_s_barrier();
    read_frags(fa0, fb0, 0, 0);

    int buf = 0;  // ring buffer of the current K step
    for (int it = 0; it < nk - 1; ++it) {
        // first half of K step `it`
        read_frags(fa1, fb1, buf, 1);
        mfma_all(fa0, fb0);
        interleave_hint(std::integral_constant<int, 0>{});
        // second half; meanwhile make stage it+1 visible and refill the buffer freed by step it-1
        const int nbuf = buf + 1 == NSTAGE ? 0 : buf + 1;
        if constexpr (!ONESHOT) {
            wait_vmcnt_imm<(NSTAGE - 3) * LPS>();
            __builtin_amdgcn_s_barrier();
            issue_stage(it + NSTAGE - 1 < nk ? it + NSTAGE - 1 : nk - 1, buf == 0 ? NSTAGE - 1 : buf - 1);
        }
        read_frags(fa0, fb0, nbuf, 0);
        mfma_all(fa1, fb1);
        interleave_hint(std::integral_constant<int, ONESHOT ? 0 : SA + SB>{});
        buf = nbuf;
    }
    // last K step
    read_frags(fa1, fb1, buf, 1);
    if (has_tail) {
        // chunk index of this lane inside the 64-byte step: kk*2 + (lane >> 5)
        const int c0 = lane >> 5, c1 = 2 + (lane >> 5);
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            if (c0 >= tail_chunks) fa0[i] = v4i{0, 0, 0, 0};
            if (c1 >= tail_chunks) fa1[i] = v4i{0, 0, 0, 0};
        }
    }
    mfma_all(fa0, fb0);
    mfma_all(fa1, fb1);
    } else if constexpr (PAIR) {
    // ---- 16x16x64 shape, pairs of steps: four waves, one per SIMD, each a quarter of the tile.  What a step costs beside its MFMAs is the
    // LDS (256 x 160, per CU and step: 52 KB of fragments and 26 KB of loads written, 610 cycles at 128 bytes a cycle against 640 of
    // MFMAs; with eight waves of half the size 72 + 26 KB, 770) and, under the power cap, the energy of moving those bytes.  A wave holds
    // the fragments of a step and reads the next step's meanwhile into a second set, so that it needs no partner on its SIMD to cover LDS
    // latency.  One barrier per pair: all of a pair is in registers when its second step begins, so behind that barrier its stage can
    // be filled again, and loads have two pairs' time to arrive.  us, eight waves / these (kernel alone): 1000 x 9216 -> 9216 row-major 87.6 /
    // 82.5, tiled 79.4 / 77.2, 512 x 5120 -> 20480 58.9 / 56.3, 512 x 20480 -> 5120 in four splits 61.8 / 59.1, 1000 x 9216 -> 9216
    // by 192 x 224 85.6 / 78.7; equal on short K (2048 x 784 -> 2048 11.7 / 12.1).  (This loop and its registers want the compiler's option
    // for MFMAs on plain vector registers; the other form copies fragments between the two register files, 30 % slower.)
    constexpr int RBT = RBA + RBB;             // 16-row blocks of a stage, A's then B's, two halves (steps) each
    constexpr int SL = RBT / NW;               // wave w fetches the blocks w, w + NW, .. whole
    constexpr bool HALF = RBT % NW != 0;       // ... and of the two left over one half
    static_assert(RBT % NW == 0 || RBT % NW == 2, "halves dealt evenly");
    constexpr int LP = 2 * SL + (HALF ? 1 : 0);  // loads of a wave per pair
    constexpr int L0 = LP / 2;                 // of pair pr + NSTAGE: issued behind the barrier in pair pr, the others in the first step of pair pr + 1
    static_assert((NSTAGE - 1) * LP <= 63, "vmcnt");
    const int steps_end = nk;  // of this split
    int8_t* const baseA = const_cast<int8_t*>(p.A) + (int64_t)m0 * p.lda;
    int8_t* const baseB = const_cast<int8_t*>(p.B) + (int64_t)n0 * p.ldb;
    auto left = [&](int rows, int64_t ld) {  // bytes from the tile's first row to the end of the operand
        const int64_t b = (TILED ? (int64_t)((rows + 15) & ~15) : (int64_t)rows) * ld;
        return (int)(b < 0x7fffffff ? b : 0x7fffffff);
    };
    const int lenA = left(p.M - m0, p.lda), lenB = left(p.N - n0, p.ldb);
    auto block_of = [&](int i) { return i < SL ? i * NW + wave : SL * NW + (wave >> 1); };
    uint32_t vo[SL + HALF];
#pragma unroll
    for (int i = 0; i < SL + HALF; ++i) {
        const int b = block_of(i), r = (b < RBA ? b : b - RBA) * 16;
        vo[i] = TILED ? (uint32_t)(r * (int)p.lda + lane * 16) : (uint32_t)((r + (lane >> 2)) * (int)p.lda + chunk * 16);  // (lda = ldb = K)
    }
    static_assert(RBA % NW == 0, "a slot is of one operand");
    // load number L of this wave for the stage of pair `pr`: both halves of a block one right after the other
    auto issue = [&](auto L_, int pr, int buf) {
        constexpr int L = decltype(L_)::value, i = L / 2;
        constexpr bool isA = i < SL && i * NW < RBA;
        const int h = i < SL ? (L & 1) : (wave & 1), st = 2 * pr + h;
        const auto rs = __builtin_amdgcn_make_buffer_rsrc(isA ? baseA : baseB, 0, st < steps_end ? (isA ? lenA : lenB) : 0, 0x00027000);
        uint32_t o = vo[i];
        if constexpr (!TILED) o |= has_tail && st == steps_end - 1 && chunk >= tail_chunks ? 0x80000000u : 0u;
        buffer_to_lds<false>(rs, smem + buf * STAGE + block_of(i) * 2048 + h * 1024, o, (kbeg + st) * KSTEP);
    };
    static_for<NSTAGE>([&](auto S_) {
        constexpr int S = decltype(S_)::value;
        static_for<(S < NSTAGE - 1 ? LP : L0)>([&](auto L_) { issue(L_, S, S); });
    });
    wait_vmcnt_imm<(NSTAGE - 2) * LP + L0>();  // pair 0 has landed
    if (PRE_RES && R) fetch_residual(0, 0);
    __builtin_amdgcn_s_barrier();
    v4i fa[2][MI], fb[2][NI];
    // read number X of a step's fragments, in the order the MFMAs want them: B 0, A 0 .. MI - 1, B 1 ..
    auto read = [&](auto X_, auto SET_, const char* sp) {
        constexpr int X = decltype(X_)::value, SET = decltype(SET_)::value;
        if constexpr (X == 0) fb[SET][0] = *(const v4i*)(sp + fragB0);
        else if constexpr (X <= MI) fa[SET][X - 1] = *(const v4i*)(sp + fragA0 + (X - 1) * FB);
        else fb[SET][X - MI] = *(const v4i*)(sp + fragB0 + (X - MI) * FB);
    };
    constexpr int NM = MI * NI, NR = MI + NI;
    static_for<NR>([&](auto X_) { read(X_, std::integral_constant<int, 0>{}, smem); });
    // Sub-step SUB of pair `pr` out of stage `buf`; `sn` is where the next step's fragments lie.  Its reads and loads are spread over the
    // MFMAs by scheduling fences: in the second step from the barrier on, which stands behind the eighth MFMA; none behind the last twelve,
    // which cover the latency of the last reads.
    auto step = [&](auto SUB_, int pr, int buf, const char* sn) {
        constexpr int SUB = decltype(SUB_)::value, BAR = 8;
        constexpr int FIRST = SUB ? BAR : 0, SPAN = NM - 12 - FIRST, NLD = SUB ? L0 : LP - L0;
        constexpr auto upto = [](int m, int n) { return m <= FIRST ? 0 : m >= FIRST + SPAN ? n : (m - FIRST) * n / SPAN; };
        static_for<NM>([&](auto M_) {
            constexpr int m = decltype(M_)::value, j = m / MI, i = m % MI;
            if constexpr (SUB == 1 && m == BAR) {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // all of this pair is in registers
                wait_vmcnt_imm<(NSTAGE - 2) * LP>();                // pair pr + 1 has landed
                __builtin_amdgcn_s_barrier();
            }
            acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[SUB][j], fa[SUB][i], acc[i][j], 0, 0, 0);
            constexpr int r0 = upto(m, NR), r1 = upto(m + 1, NR), l0 = upto(m, NLD), l1 = upto(m + 1, NLD);
            if constexpr (r1 > r0 || l1 > l0) {
                __builtin_amdgcn_sched_barrier(0);
                static_for<r1 - r0>([&](auto D_) { read(std::integral_constant<int, r0 + decltype(D_)::value>{}, std::integral_constant<int, 1 - SUB>{}, sn); });
                static_for<l1 - l0>([&](auto D_) {
                    constexpr int L = l0 + decltype(D_)::value;
                    if constexpr (SUB) issue(std::integral_constant<int, L>{}, pr + NSTAGE, buf);
                    else issue(std::integral_constant<int, L0 + L>{}, pr - 1 + NSTAGE, buf == 0 ? NSTAGE - 1 : buf - 1);
                });
                __builtin_amdgcn_sched_barrier(0);
            }
        });
    };
    const int npairs = (nk + 1) >> 1;
    int buf = 0;
    for (int pr = 0; pr < npairs; ++pr) {
        const int nbuf = buf + 1 == NSTAGE ? 0 : buf + 1;
        step(std::integral_constant<int, 0>{}, pr, buf, smem + buf * STAGE + 1024);
        step(std::integral_constant<int, 1>{}, pr, buf, smem + nbuf * STAGE);
        buf = nbuf;
    }
    } else {
    // ---- 16x16x64 shape.  A wave owns 64 rows x WN columns.  Its four A fragments of a K step stay in registers for the
    // whole step (the next step's four are read meanwhile into a second set); the NI B fragments come in NP parts of
    // two, double buffered: while the 8 MFMAs of a part issue, the two fragments of the next part are read.
    // Per step 4 + NI reads of 1 KB and 4 NI MFMAs.  The barrier that publishes stage it + 1 sits in front of the third
    // part from the end; the reads that belong to the next step (its A fragments, its first part of B) come after it.
    constexpr int NQ = 2, NP = NI / NQ, PB = NP - 3;
    static_assert(PB >= 0, "parts of a K step");
    v4i fa[2][MI], fbq[2][NQ];
#pragma unroll
    for (int s = 0; s < NSTAGE - 1; ++s) issue_stage(s < nk ? s : nk - 1, s);
    wait_vmcnt_imm<(NSTAGE - 2) * LPS>();
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int i = 0; i < MI; ++i) fa[0][i] = *(const v4i*)(smem + fragA0 + i * 1024);
#pragma unroll
    for (int k = 0; k < NQ; ++k) fbq[0][k] = *(const v4i*)(smem + fragB0 + k * 1024);

    // Every step is the same code: the last one also reads "next" fragments (from a buffer that holds an old stage:
    // valid LDS, values never used) and refills a buffer nobody reads.  The host sends only K ranges of an even number
    // of whole steps here (K % 128 == 0, no K split), so the loop runs in pairs and there is no second copy of the step
    // outside it (with one, the register allocation of the epilogue spilled hundreds of registers per lane).
    // P0: which of the two B fragment sets the step's first part finds filled (with an odd number of parts per step the
    // two steps of the unrolled pair start on different sets).
    auto step = [&](auto P0_, v4i(&cur)[MI], v4i(&nxt)[MI], int it, int buf) {
        constexpr int P0 = decltype(P0_)::value;
        const int nbuf = buf + 1 == NSTAGE ? 0 : buf + 1;
        const char* sb = smem + buf * STAGE + fragB0;
        const char* sn = smem + nbuf * STAGE;
        // the stage this step fetches (past the end of the K range the last one again), into the buffer of step it - 1
        const int kt = it + NSTAGE - 1 < nk ? it + NSTAGE - 1 : nk - 1;
        const int8_t* ga = Ab + (int64_t)kt * KSTEP;
        const int8_t* gb = Bb + (int64_t)kt * KSTEP;
        char* refill = smem + (buf == 0 ? NSTAGE - 1 : buf - 1) * STAGE;
        static_for<NP>([&](auto Q_) {
            constexpr int q = decltype(Q_)::value;
            if constexpr (q == PB) {
                wait_vmcnt_imm<(NSTAGE - 3) * LPS>();
                __builtin_amdgcn_s_barrier();
            }
            // next step's A fragments: two each in the last two parts.  (None in the first part behind the barrier: there
            // the eight waves run in step and their stage loads and reads meet in the LDS; with two of the four reads
            // there the whole step took an eighth longer.)
            constexpr int pa = q - PB;  // parts behind the barrier so far
            constexpr int an0 = pa <= 1 ? 0 : 2;
            constexpr int an_cnt = pa <= 0 ? 0 : 2;
            // The part in the instruction stream, fixed by scheduling fences: its first MFMA (in front of it the wait
            // for this part's fragments, which is exact there: nothing younger is in flight), then the reads of the
            // next part and, behind the barrier, the stage's global->LDS loads, then the other seven MFMAs, which
            // cover the latency of those reads.
            acc[0][q * NQ] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fbq[(q + P0) & 1][0], cur[0], acc[0][q * NQ], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (q >= PB) {
                // the stage's loads (the first SA are A blocks, the others B blocks), spread over the parts behind the
                // barrier: issued in one burst they cost an eighth more time per step
                constexpr int per = (LPS + NP - PB - 1) / (NP - PB), i0 = (q - PB) * per, i1 = i0 + per < LPS ? i0 + per : LPS;
                static_for<(i1 > i0 ? i1 - i0 : 0)>([&](auto D_) {
                    constexpr int i = i0 + decltype(D_)::value;
                    // (the offset is made opaque here so that its widening to 64 bits stays next to the load: hoisted out
                    // of the loop it costs a register pair per load and the scalar-base addressing form)
                    uint32_t o = i < SA ? offA[i < SA ? i : 0] : offB[i < SA ? 0 : i - SA];
                    asm volatile("" : "+v"(o));
                    if constexpr (i < SA) __builtin_amdgcn_global_load_lds(GPTR(ga + o), LPTR(refill + ldsA[i]), 16, 0, 0);
                    else __builtin_amdgcn_global_load_lds(GPTR(gb + o), LPTR(refill + ldsB[i - SA]), 16, 0, 0);
                });
            }
            if constexpr (q < NP - 1) {
#pragma unroll
                for (int k = 0; k < NQ; ++k) fbq[(q + 1 + P0) & 1][k] = *(const v4i*)(sb + ((q + 1) * NQ + k) * 1024);
            } else {
#pragma unroll
                for (int k = 0; k < NQ; ++k) fbq[(q + 1 + P0) & 1][k] = *(const v4i*)(sn + fragB0 + k * 1024);
            }
            static_for<an_cnt>([&](auto K_) {
                constexpr int k = an0 + decltype(K_)::value;
                nxt[k] = *(const v4i*)(sn + fragA0 + k * 1024);
            });
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < NQ; ++k)
#pragma unroll
                for (int i = 0; i < MI; ++i)
                    if (k + i > 0)
                        acc[i][q * NQ + k] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fbq[(q + P0) & 1][k], cur[i], acc[i][q * NQ + k], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    int buf = 0;
    for (int it = 0; it < nk; it += 2) {
        step(std::integral_constant<int, 0>{}, fa[0], fa[1], it, buf);
        buf = buf + 1 == NSTAGE ? 0 : buf + 1;
        step(std::integral_constant<int, NP & 1>{}, fa[1], fa[0], it + 1, buf);
        buf = buf + 1 == NSTAGE ? 0 : buf + 1;
    }
    }
    wait_vmcnt_imm<0>();  // the refills issued past the end of the K range have landed
    if constexpr (PAIR && EPI == EPI_I32 && MI * NI * AV >= 160) {
        // A zero the compiler cannot see through, added to the sums: with stores alone behind the loop it keeps some of them in the accumulation registers
        // and copies fragments between the two files in every step (256 x 160 tiled 26 copies a pair: 1000 x 9216 -> 9216 82.9 us, so 80.2).
        int zero;
        asm volatile("s_mov_b32 %0, 0" : "=s"(zero));
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int e = 0; e < AV; ++e) acc[i][j][e] += zero;
    }

    // ---- epilogue.  Accumulator block (i, j) is the transposed 32x32 output block: lane l, register v
    // holds output row (l & 31), column 8*(v/4) + 4*(l >> 5) + (v & 3) of the block, i.e. registers
    // 4g .. 4g+3 are four neighbouring columns of one row.  (16x16 blocks: row (l & 15), columns 4*(l >> 4) + v.)
    const int row_l = lane & (MF - 1), col_l = (lane >> (MF == 32 ? 5 : 4)) * 4;
    if constexpr (EPI == EPI_I32) {
        int32_t* out = p.acc_out + ((int64_t)split * p.M) * p.N;
        const bool vec4 = (p.N & 3) == 0;  // 16-byte stores stay aligned and inside the row
        if constexpr (PAIR) {
            // One wave per SIMD: nothing covers what stands between two stores, so no branches and no 64-bit addresses; the buffer's length bounds the
            // rows, an offset beyond any length the columns (N < 2^20: the offsets of 256 rows end below that).  us, with a bounds check and an address each /
            // so: 1966 x 320 -> 968 row-major 10.1 / 9.6, 749 x 608 -> 6680 12.5 / 12.2, 960 x 624 -> 3992 12.0 / 11.7.
            if (vec4 && p.N < (1 << 20)) {
                const int64_t left = (int64_t)(p.M - m0) * p.N * 4;
                const auto rc = __builtin_amdgcn_make_buffer_rsrc(out + (int64_t)m0 * p.N, 0, (int)(left < 0x7fffffff ? left : 0x7fffffff), 0x00027000);
                uint32_t vo[NI];
#pragma unroll
                for (int j = 0; j < NI; ++j) {
                    const int col = n0 + wn * WN + j * MF + col_l;
                    vo[j] = col < p.N ? (uint32_t)((wm * WM + row_l) * p.N + col) * 4u : 0x80000000u;
                }
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int j = 0; j < NI; ++j)
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, acc[i][j]), rc, (int)(vo[j] + (uint32_t)(i * MF * 4) * (uint32_t)p.N), 0, 0);
                return;
            }
        }
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int row = m0 + wm * WM + i * MF + row_l;
            if (row < p.M) {
#pragma unroll
                for (int j = 0; j < NI; ++j)
#pragma unroll
                    for (int g = 0; g < QG; ++g) {
                        const int col = n0 + wn * WN + j * MF + 8 * g + col_l;
                        int32_t* dst = out + (int64_t)row * p.N + col;
                        if (vec4 && col < p.N) {
                            *(v4i*)dst = v4i{acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
                        } else {
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                if (col + e < p.N) dst[e] = acc[i][j][4 * g + e];
                        }
                    }
            }
        }
    } else {
        // The 16-bit tile is staged in LDS (free once the K loop is over) so that global memory is
        // written in whole 512-byte row segments, 16 bytes per lane, instead of 2-byte scatters; the
        // residual tile is fetched the same way.  Row pitch +16 B keeps the two half-waves (4 rows
        // apart) on different banks.
        constexpr int PITCH = BN * 2 + 16;
        static_assert(GR * PITCH <= SMEM_BYTES && GR % 32 == 0, "epilogue staging must fit in the LDS allocation");
        uint16_t* C = (uint16_t*)p.C + (int64_t)batch * p.strideC;
        float* const sv_col = (float*)(smem + EPI_VEC);
        float* const sv_bias = sv_col + BN;
        float* const sv_row = sv_bias + BN;
        if constexpr (!PRE) fetch_scales();
        // Accumulators to fp32 in place, before anything else of the epilogue: the conversion does not depend on the
        // row group or on the optional terms, so the compiler moves it in front of the loop and the switch below
        // anyway, and into new registers if left to itself (the 384-wide tile then spilled thirty per lane).
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                typedef float accf_t __attribute__((ext_vector_type(AV)));
                acc[i][j] = __builtin_bit_cast(acc_t, __builtin_convertvector(acc[i][j], accf_t));
            }
        float rq = 0.0f;
        if constexpr (EPI == EPI_CODES) {
            const float delta = p.q8_step[0];
            rq = delta > 0.0f ? 1.0f / delta : 0.0f;
        }
        // Rows that are not whole 16-byte pieces: between memory and LDS in aligned pieces of W neighbouring values (N % 4 == 0: four, else two), so that
        // neighbouring lanes share lines, several pieces in flight; an odd N eight values a thread, one by one.  IN: the residual, of which what lies
        // outside is some other value (loads under a condition are waited for one by one; nobody reads it).  us, eight values a thread one by one / so, with a
        // residual: 530 x 2304 -> 17220 tiled 53.0 / 34.3, 222 x 2400 -> 21958 row-major 48.9 / 40.6.
        auto ragged = [&](auto W_, auto IN_, int g0, int opaque0) {
            constexpr int W = decltype(W_)::value, PW = W == 1 ? 8 : W, CW = BN / PW, ALL = GR * CW, U = W == 1 ? 2 : 8;
            typedef uint32_t piece __attribute__((ext_vector_type(PW / 2)));
#pragma unroll 1
            for (int k0 = 0; k0 < (ALL + NW * 64 - 1) / (NW * 64); k0 += U) {
                uint16_t one[U][W == 1 ? 8 : 1];
                piece val[U];
                auto place = [&](int k, int& r, int& c) {
                    const int q = (int)threadIdx.x + opaque0 + (k0 + k) * NW * 64;
                    r = q / CW;
                    c = (q - r * CW) * PW;
                    return ALL % (U * NW * 64) == 0 || q < ALL;
                };
#pragma unroll
                for (int k = 0; k < U; ++k) {
                    int r, c;
                    const bool there = place(k, r, c);
                    if constexpr (decltype(IN_)::value) {
                        const int row = m0 + g0 + r < p.M ? m0 + g0 + r : p.M - 1, col = n0 + c;
                        const uint16_t* src = R + (int64_t)row * p.N;
                        if constexpr (W == 1) {
#pragma unroll
                            for (int t = 0; t < 8; ++t) one[k][t] = src[col + t < p.N ? col + t : p.N - 1];
                        } else {
                            val[k] = *(const piece*)(src + (col < p.N ? col : 0));
                        }
                    } else if (there) {
                        val[k] = *(const piece*)(smem + r * PITCH + c * 2);
                    }
                }
#pragma unroll
                for (int k = 0; k < U; ++k) {
                    int r, c;
                    const bool there = place(k, r, c);
                    const int row = m0 + g0 + r, col = n0 + c;
                    if constexpr (decltype(IN_)::value) {
                        if constexpr (W == 1) {
#pragma unroll
                            for (int t = 0; t < 4; ++t) val[k][t] = (uint32_t)one[k][2 * t] | ((uint32_t)one[k][2 * t + 1] << 16);
                        }
                        if (there) *(piece*)(smem + r * PITCH + c * 2) = val[k];
                    } else if (there && row < p.M && col < p.N) {
                        uint16_t* dst = C + (int64_t)row * p.N + col;
                        if constexpr (W == 1) {
#pragma unroll
                            for (int t = 0; t < 8; ++t)
                                if (col + t < p.N) dst[t] = (uint16_t)(val[k][t >> 1] >> ((t & 1) * 16));
                        } else {
                            *(piece*)dst = val[k];
                        }
                    }
                }
            }
        };
#pragma unroll
        for (int eg = 0; eg < EG; ++eg) {
        const int g0 = eg * GR;  // first tile row of this group
        // A zero the compiler cannot see through, added to the row and column offsets below: without it every index,
        // bounds predicate and LDS address of all variants of phase1 counts as independent of the row group and
        // is computed in front of this loop, where some ninety such values stay live next to the accumulators.
        int opaque0;
        asm volatile("s_mov_b32 %0, 0" : "=s"(opaque0));
        __syncthreads();  // operand reads (first group) or the previous group's stores out of LDS are done
        if (eg == 0) {
            const int t = (int)threadIdx.x;
            if (t < BN) {
                sv_col[t] = col_scale;
                sv_bias[t] = col_bias;
            }
            if (t < BM) sv_row[t] = row_scale;
        }
        if (R) {
            if constexpr (WHOLE) {
#pragma unroll 1
                for (int k0 = 0; k0 < RCH; k0 += RG) {
                    if constexpr (!PRE_RES) fetch_residual(g0, k0);
#pragma unroll
                    for (int k = 0; k < RG; ++k) {
                        const int q = (int)threadIdx.x + (k0 + k) * NW * 64, r = q / CPR;
                        if (q < GR * CPR) *(v4u*)(smem + r * PITCH + (q - r * CPR) * 16) = rpre[k];
                    }
                }
            } else if ((p.N & 3) == 0) ragged(std::integral_constant<int, 4>{}, std::true_type{}, g0, opaque0);
            else if ((p.N & 1) == 0) ragged(std::integral_constant<int, 2>{}, std::true_type{}, g0, opaque0);
            else ragged(std::integral_constant<int, 1>{}, std::true_type{}, g0, opaque0);
        }
        __syncthreads();
        // The optional terms are compile-time flags inside the loop (one uniform switch outside) so the
        // common cases cost two multiplies + round per element and one 8-byte LDS write per four.  Scales and biases come from LDS, once per
        // column block: read from memory where they are used, with a bounds check each and again for every row block, they were most
        // of the 3.8 us (6.4 with a step per channel, now 1.3 and 1.3) that this part of the 256 x 160 tile took.
        auto phase1 = [&](auto HB, auto RL, auto HR, auto PC) {
            constexpr bool has_bias = decltype(HB)::value, relu = decltype(RL)::value, has_res = decltype(HR)::value, per_col = decltype(PC)::value;
            typedef float v4f __attribute__((ext_vector_type(4)));
            float xr[MI];
#pragma unroll
            for (int i = 0; i < MI; ++i) xr[i] = sv_row[wm * WM + i * MF + row_l + opaque0];
            if constexpr (!per_col) {  // one scale for all columns
                const float ws = sv_col[opaque0];
#pragma unroll
                for (int i = 0; i < MI; ++i) xr[i] = xr[i] * ws;
            }
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int g = 0; g < QG; ++g) {
                    const int lcol = wn * WN + j * MF + 8 * g + col_l + opaque0;
                    v4f wv;
                    if constexpr (per_col) wv = *(const v4f*)(sv_col + lcol);
                    v4f bv = {0.0f, 0.0f, 0.0f, 0.0f};
                    if constexpr (has_bias) bv = *(const v4f*)(sv_bias + lcol);
#pragma unroll
                    for (int i = 0; i < MI; ++i) {
                        if (EG > 1 && (wm * WM + i * MF) / GR != eg) continue;  // rows of another group
                        const int lrow = wm * WM + i * MF + row_l - g0 + opaque0;
                        v2u* slot = (v2u*)(smem + lrow * PITCH + lcol * 2);
                        v2u rb = {0u, 0u};
                        if constexpr (has_res) rb = *slot;
                        auto fa = [&](int e) {
                            const int bits = acc[i][j][4 * g + e];  // a copy: a vector element is no object to cast from
                            return __builtin_bit_cast(float, bits);
                        };
                        auto c = [&](int e) { return per_col ? xr[i] * wv[e] : xr[i]; };
                        const uint32_t o01 = dequant_pair_f<BF16>(fa(0), fa(1), c(0), c(1), bv[0], bv[1], has_bias, relu, rb[0], has_res);
                        const uint32_t o23 = dequant_pair_f<BF16>(fa(2), fa(3), c(2), c(3), bv[2], bv[3], has_bias, relu, rb[1], has_res);
                        *slot = v2u{o01, o23};
                    }
                    if constexpr (FULL) __builtin_amdgcn_sched_barrier(0);  // (or the LDS reads of all column blocks are moved up here)
                }
        };
        using T_ = std::true_type;
        using F_ = std::false_type;
        auto with = [&](auto PC) {
            switch ((p.bias ? 1 : 0) | (p.relu ? 2 : 0) | (R ? 4 : 0)) {
                case 0: phase1(F_{}, F_{}, F_{}, PC); break;
                case 1: phase1(T_{}, F_{}, F_{}, PC); break;
                case 2: phase1(F_{}, T_{}, F_{}, PC); break;
                case 3: phase1(T_{}, T_{}, F_{}, PC); break;
                case 4: phase1(F_{}, F_{}, T_{}, PC); break;
                case 5: phase1(T_{}, F_{}, T_{}, PC); break;
                case 6: phase1(F_{}, T_{}, T_{}, PC); break;
                default: phase1(T_{}, T_{}, T_{}, PC); break;
            }
        };
        if (p.w_per_channel) with(T_{});
        else with(F_{});
        __syncthreads();
        if constexpr (EPI == EPI_CODES) {
            // int8 output (N % 8 == 0): a thread quantizes W neighbouring 16-bit values, 16 (one chunk of the tiled layout, 16 bytes of a row) or,
            // where rows are not whole 16-byte pieces, 8.  Tiled codes leave in the order of the 1 KB blocks, 32 columns of 16 rows after the
            // other where the tile is not whole blocks wide.  What counts is LDS latency: eight codes a trip, with an index division, a read
            // and its wait each, took 300 x 4096 -> 16384 tiled 36.2 us (now 33.6; 16-bit values 32.0), 512 x 2048 -> 8192 20.1 (18.0; 17.5).
            auto store_codes = [&](auto W_, bool tiled_codes) {
                constexpr int W = decltype(W_)::value, CQ = BN / W, ALL = GR * CQ, QCH = (ALL + NW * 64 - 1) / (NW * 64);
                constexpr int SG = FULL ? 1 : QCH < 4 ? QCH : QCH % 5 == 0 ? 5 : QCH % 4 == 0 ? 4 : QCH % 3 == 0 ? 3 : 4;  // pieces a thread has in flight out of LDS
                auto place = [&](int q, int& r, int& c) {
                    if (W == 16 && tiled_codes) {
                        constexpr int CB = BN % 64 == 0 ? 4 : 2;  // chunks of a row that go out together
                        static_assert(BN % 32 == 0 && GR % 16 == 0, "whole groups of chunks");
                        const int strip = q / (16 * CQ), in = q - strip * (16 * CQ);
                        r = strip * 16 + in / CB % 16;
                        c = (in / (16 * CB) * CB + in % CB) * W;
                    } else {
                        r = q / CQ;
                        c = (q - r * CQ) * W;
                    }
                };
#pragma unroll 1
                for (int k0 = 0; k0 < QCH; k0 += SG) {
                    v4u val[SG][W / 8];
#pragma unroll
                    for (int k = 0; k < SG; ++k) {
                        const int q = (int)threadIdx.x + (k0 + k) * NW * 64;
                        int r, c;
                        place(q, r, c);
                        if (ALL % (SG * NW * 64) == 0 || q < ALL) {
#pragma unroll
                            for (int h = 0; h < W / 8; ++h) val[k][h] = *(const v4u*)(smem + r * PITCH + c * 2 + h * 16);
                        }
                    }
#pragma unroll
                    for (int k = 0; k < SG; ++k) {
                        const int q = (int)threadIdx.x + (k0 + k) * NW * 64;
                        int r, c;
                        place(q, r, c);
                        const int row = m0 + g0 + r, col = n0 + c;
                        if ((ALL % (SG * NW * 64) == 0 || q < ALL) && row < p.M && col < p.N) {
                            uint32_t w[W / 4];  // (clamp + add of 1.5 * 2^23: the code in the low byte, the same integer as requant_code's rint + clamp)
#pragma unroll
                            for (int t = 0; t < W / 4; ++t) {
                                const uint32_t lo = val[k][t >> 1][(t & 1) * 2], hi = val[k][t >> 1][(t & 1) * 2 + 1];
                                w[t] = pack4_low_bytes(code_bits(load16_bits<BF16>(lo) * rq), code_bits(load16_bits<BF16>(lo >> 16) * rq),
                                                       code_bits(load16_bits<BF16>(hi) * rq), code_bits(load16_bits<BF16>(hi >> 16) * rq));
                            }
                            int8_t* dst = code_dst(p.q8_out, row, col, p.N, W == 16 && tiled_codes);
                            if constexpr (W == 16) *(v4u*)dst = v4u{w[0], w[1], w[2], w[3]};
                            else *(v2u*)dst = v2u{w[0], w[1]};
                        }
                    }
                }
            };
            if ((p.N & 15) == 0) store_codes(std::integral_constant<int, 16>{}, p.q8_tiled != 0);
            else store_codes(std::integral_constant<int, 8>{}, false);
        } else if constexpr (WHOLE) {
            constexpr int SG = FULL ? 2 : RCH % 5 == 0 ? 5 : RCH % 4 == 0 ? 4 : RCH % 3 == 0 ? 3 : 4;  // pieces a thread has in flight out of LDS
#pragma unroll 1
            for (int k0 = 0; k0 < RCH; k0 += SG) {
                v4u val[SG];
#pragma unroll
                for (int k = 0; k < SG; ++k) {
                    const int q = (int)threadIdx.x + (k0 + k) * NW * 64, r = q / CPR;
                    if (GR * CPR % (SG * NW * 64) == 0 || q < GR * CPR) val[k] = *(const v4u*)(smem + r * PITCH + (q - r * CPR) * 16);
                }
#pragma unroll
                for (int k = 0; k < SG; ++k) {
                    const int q = (int)threadIdx.x + (k0 + k) * NW * 64, r = q / CPR, row = m0 + g0 + r, col = n0 + (q - r * CPR) * 8;
                    if ((GR * CPR % (SG * NW * 64) == 0 || q < GR * CPR) && row < p.M && col < p.N)
                        __builtin_nontemporal_store(val[k], (v4u*)(C + (int64_t)row * p.N + col));
                }
            }
        } else if ((p.N & 3) == 0) ragged(std::integral_constant<int, 4>{}, std::false_type{}, g0, opaque0);
        else if ((p.N & 1) == 0) ragged(std::integral_constant<int, 2>{}, std::false_type{}, g0, opaque0);
        else ragged(std::integral_constant<int, 1>{}, std::false_type{}, g0, opaque0);
        }  // row groups
    }
}

template <int EPI, bool BF16, bool TILED>
void launch_cfg(const TilePlan& pl, const GemmArgs& a, int batch, hipStream_t st)
{
    constexpr int LAY = TILED ? LAY_TILED : LAY_ROWS;
    dim3 grid((unsigned)(pl.tiles_m * pl.tiles_n * pl.splits), (unsigned)batch);
#define SQ_LAUNCH_MF(BM, BN, WGM, WGN, NST, MF)                                                                   \
    do {                                                                                                          \
        sq_launch((gemm_i8_kernel<BM, BN, WGM, WGN, NST, EPI, BF16, LAY, 1, false, MF>), grid, dim3(WGM * WGN * 64), 0, st, a); \
    } while (0)
#define SQ_LAUNCH_PAIR(BM, BN) sq_launch((gemm_i8_kernel<BM, BN, 2, 2, 3, EPI, BF16, LAY, 1, false, 16, true>), grid, dim3(256), 0, st, a)
#define SQ_LAUNCH(BM, BN, WGM, WGN, NST) SQ_LAUNCH_MF(BM, BN, WGM, WGN, NST, 32)
    switch (pl.cfg) {
        case 0: SQ_LAUNCH(256, 256, 2, 4, 4); break;
        case 1: SQ_LAUNCH(128, 256, 1, 4, 6); break;
        case 2: SQ_LAUNCH(64, 256, 1, 4, 7); break;
        case 3: SQ_LAUNCH(32, 256, 1, 4, 8); break;
        case 6: SQ_LAUNCH(256, 192, 4, 2, 4); break;
        case 9: SQ_LAUNCH(256, 384, 2, 4, 4); break;
        case 10: SQ_LAUNCH_MF(256, 256, 4, 2, 4, 16); break;
        case 11: SQ_LAUNCH_MF(256, 384, 4, 2, 4, 16); break;
        case 12: SQ_LAUNCH_MF(256, 192, 4, 2, 5, 16); break;
        case 13: SQ_LAUNCH_PAIR(256, 160); break;
        case 14: SQ_LAUNCH_PAIR(256, 128); break;
        case 15: SQ_LAUNCH_PAIR(192, 224); break;
        case 16: SQ_LAUNCH_PAIR(192, 160); break;
        case 8:
            sq_launch((gemm_i8_kernel<128, 128, 2, 2, 3, EPI, BF16, LAY, 4, true>), grid, dim3(256), 0, st, a);
            break;
        case 7:
            sq_launch((gemm_i8_kernel<128, 128, 2, 2, 3, EPI, BF16, LAY, 3>), grid, dim3(256), 0, st, a);
            break;
    }
#undef SQ_LAUNCH
#undef SQ_LAUNCH_MF
#undef SQ_LAUNCH_PAIR
}

template <bool TILED> void tile_launch(const TilePlan& pl, const GemmArgs& a, bool to_i32, bool bf16, int batch, hipStream_t st)
{
    if (to_i32) launch_cfg<EPI_I32, false, TILED>(pl, a, batch, st);
    else if (bf16) launch_cfg<EPI_DEQUANT, true, TILED>(pl, a, batch, st);
    else launch_cfg<EPI_DEQUANT, false, TILED>(pl, a, batch, st);
}
template <bool TILED> void tile_launch_ragged(const TilePlan& pl, const GemmArgs& a, bool bf16, int batch, hipStream_t st)
{
    if (bf16) launch_cfg<EPI_RAGGED, true, TILED>(pl, a, batch, st);
    else launch_cfg<EPI_RAGGED, false, TILED>(pl, a, batch, st);
}
template <bool TILED> void tile_launch_codes(const TilePlan& pl, const GemmArgs& a, bool bf16, hipStream_t st)
{
    if (bf16) launch_cfg<EPI_CODES, true, TILED>(pl, a, 1, st);
    else launch_cfg<EPI_CODES, false, TILED>(pl, a, 1, st);
}

}  // namespace
