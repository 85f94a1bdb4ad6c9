// P V of attention (sq_w8a8_bmm, trans_b = 0): C = (A B) * alpha with A [m, k] int8 codes row-major and B [k, n] int8, n contiguous, per
// batch entry; 16-bit output.
//
// What bounds it is the stream of A (k bytes per row against n 16-bit outputs, B shared by a head's rows).  So A goes from memory straight
// into MFMA operand registers, whole 128-byte lines at a time (two 64-byte K steps requested one after the other), two stages ahead; no LDS
// and no barrier on its way.  B's rows travel to LDS as they lie (16-byte columns permuted where the row pitch would put the rows of a
// read on the same banks), three stages of 128 keys, one barrier per stage; the LDS transpose read
// (ds_read_b64_tr_b8: sixteen lanes name the halves of eight rows' 16 columns, lane i receives column i of them) hands them to the
// v_mfma_i32_16x16x64_i8 as they are, sixteen columns at a time: no columns are computed that are not there.
// us by graph replay, operands from memory; a 256 x 128 LDS-staged tile with the transposition in registers / this: 128 heads x 1024^2 x 80
// 48.8 / 38.4, x 128 48.8 / 42.8, 256 x 1024^2 x 112 81.8 / 68.1, 199 x 448^2 x 96 26.9 / 15.0, 12 x 64^2 x 80 7.7 / 3.1, 768 x 2048^2 x 128
// 824 / 715.  With one column block the first takes 29 us (4.8 TB/s): the rest is LDS reads and MFMAs that do not overlap with the stream.
// A fifth wave that only loads B, or 256 bytes of a row at a time: 41-42 us; the compiler's own transpose reads: see lds_read_tr.
#include "gemm_args.h"

namespace {

constexpr int PV_KC = 128;     // keys per stage
constexpr int PV_STAGES = 3;

// NB: 16-column blocks of a workgroup; MB: 16-row blocks of a wave (four of them).  Workgroups per compute unit: three or four, with MB = 4 two (208 to 256
// registers).
template <bool BF16, int NB, int MB>
__global__ __launch_bounds__(256, MB == 4 ? 2 : NB <= 6 ? 4 : 3) void pv_kernel(const GemmArgs p)
{
    constexpr int N = NB * 16, VST = PV_KC * N, LPS = VST / 1024;
    constexpr int PITCH = N * 2 + 16, STG = 16 * MB * PITCH;
    constexpr int RING = PV_STAGES * VST, SMEM = RING > 4 * STG ? RING : 4 * STG;
    __shared__ __attribute__((aligned(1024))) char smem[SMEM];
    // position of a 16-byte column block in its LDS row: j ^ swz(key), so that eight consecutive rows of a transpose read (eight of the
    // 128-byte row pitch, four of the 64-byte one, would meet on a bank) lie apart; other pitches spread them by themselves
    auto swz = [](int key) { return NB == 8 ? (key >> 1) & 3 : NB == 4 ? (key >> 2) & 1 : 0; };

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // XCD-aware order over (batch, tile): an XCD works through whole heads, whose row blocks share B in its L2
    const int64_t total = (int64_t)gridDim.x * gridDim.y, wg = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    const int64_t per = total >> 3;
    const int xcd = (int)(wg & 7), rest = (int)(total & 7);
    const int64_t pid = xcd * per + (xcd < rest ? xcd : rest) + (wg >> 3);
    int batch, t;
    if (total < ((int64_t)1 << 31)) {
        batch = (int)((uint32_t)pid / gridDim.x);
        t = (int)((uint32_t)pid - (uint32_t)batch * gridDim.x);
    } else {
        batch = (int)(pid / gridDim.x);
        t = (int)(pid - (int64_t)batch * gridDim.x);
    }
    const int tm = p.tiles_n == 1 ? t : t / p.tiles_n, n0 = p.tiles_n == 1 ? 0 : (t - tm * p.tiles_n) * N;
    const int m0 = tm * (64 * MB);
    const int nst = (p.K + PV_KC - 1) / PV_KC;

    // ---- B: stage s of 128 rows, 1 KB per load, dealt to the waves; what lies past the last row arrives as zeros (columns past n: whatever
    // follows, their results are not stored)
    int8_t* const Bb = const_cast<int8_t*>(p.B) + (int64_t)batch * p.strideB + n0;
    constexpr int NV = LPS / 4, NV1 = (LPS + 3) / 4;  // loads of a wave per stage, fewest and most
    auto load_b = [&](int s) {
        char* const dst = smem + s % PV_STAGES * VST;
        const int64_t at = (int64_t)s * PV_KC * p.N, left = (int64_t)p.K * p.N - n0 - at;
        const auto rs = __builtin_amdgcn_make_buffer_rsrc(Bb + at, 0, left <= 0 ? 0 : (int)(left < 0x7fffffff ? left : 0x7fffffff), 0x00027000);
#pragma unroll
        for (int i = 0; i < NV1; ++i) {
            if (i == NV && wave >= LPS % 4) break;
            const int c = (i * 4 + wave) * 64 + lane, key = c / NB, j = (c - key * NB) ^ swz(key);
            buffer_to_lds<false>(rs, dst + (i * 4 + wave) * 1024, (uint32_t)(key * p.N + j * 16), 0);
        }
    };

    // ---- this wave: rows w0 .. w0 + 16 MB - 1, all N columns.  Operand of rows: lane l feeds row (l & 15) with the 16 bytes at 16 (l >> 4)
    // of a 64-byte step; what lies outside A (rows past m, bytes past k) arrives as zeros.
    const int w0 = m0 + wave * (16 * MB), g = lane >> 4, r16 = lane & 15;
    const int rows = p.M - w0 < 16 * MB ? p.M - w0 : 16 * MB;
    const auto ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(p.A) + (int64_t)batch * p.strideA + (rows > 0 ? (int64_t)w0 * p.lda : 0), 0,
                                                      rows > 0 ? rows * (int)p.lda : 0, 0x00027000);
    uint32_t ao[MB];
#pragma unroll
    for (int i = 0; i < MB; ++i) ao[i] = (uint32_t)((i * 16 + r16) * (int)p.lda + g * 16);
    v4i pa[2][MB][2];
    auto load = [&](auto SET_, int s) {
        constexpr int SET = decltype(SET_)::value;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int k0 = s * PV_KC + h * 64;
            const uint32_t out = k0 + g * 16 < p.K ? 0u : 0x80000000u;
#pragma unroll
            for (int i = 0; i < MB; ++i)
                pa[SET][i][h] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(ra, (int)((ao[i] + (uint32_t)k0) | out), 0, 0));
        }
    };
    // Operand of columns: lane l feeds column (l & 15) of a block with keys 16 (l >> 4) .. + 15 of the step: two transpose reads of eight keys
    const int vo = (16 * g + (r16 >> 1)) * N + swz(r16 >> 1) * 16 + (r16 & 1) * 8;
    v4i acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = v4i{0, 0, 0, 0};
    auto compute = [&](auto SET_, int slot) {
        constexpr int SET = decltype(SET_)::value;
        const uint32_t st = lds_address(smem + slot * VST);
        // (the row pitches with a permutation are powers of two: the column block's bits are clear in key * N)
        auto at = [&](int v, int j) { return st + (uint32_t)(NB == 8 || NB == 4 ? v ^ (j * 16) : v + j * 16); };
        static_for<2>([&](auto H_) {
            constexpr int h = decltype(H_)::value, O = h * 64 * N;
            constexpr int GROUPS = (NB + 3) / 4;  // up to four column blocks' reads under one wait
            static_for<GROUPS>([&](auto G_) {
                constexpr int j = decltype(G_)::value * NB / GROUPS, JN = (decltype(G_)::value + 1) * NB / GROUPS - j;
                uint32_t p[JN];
#pragma unroll
                for (int q = 0; q < JN; ++q) p[q] = at(vo, j + q);
                v2i r[2 * JN];
                lds_read_tr<O, O + 8 * N>(p, r);  // (the rows 8 further on have the same permutation)
#pragma unroll
                for (int q = 0; q < JN; ++q) {
                    const v4i v = {r[2 * q].x, r[2 * q].y, r[2 * q + 1].x, r[2 * q + 1].y};
#pragma unroll
                    for (int i = 0; i < MB; ++i) acc[i][j + q] = __builtin_amdgcn_mfma_i32_16x16x64_i8(v, pa[SET][i][h], acc[i][j + q], 0, 0, 0);
                }
            });
        });
    };
    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;
    // Loads in this order: none passes an asm statement that clobbers memory.  (Past the end of k zeros arrive, without traffic: loads
    // under a condition would make the compiler wait for all there might be, and copies of the stage without them spill.)
    auto fence = [] { asm volatile("" ::: "memory"); };
    load_b(0);
    fence();
    load(S0{}, 0);
    fence();
    load_b(1);
    fence();
    load(S1{}, 1);
    int slot = 0;
    auto stage = [&](auto SET_, int s) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        wait_vmcnt_imm<2 * MB + NV>();  // this wave's loads of stage s have landed; those of stage s + 1, issued since the last barrier, may be under way
        __builtin_amdgcn_s_barrier();   // ... everybody's have, and everybody is done with stage s - 1
        load_b(s + 2);
        compute(SET_, slot);
        load(SET_, s + 2);
        slot = slot == PV_STAGES - 1 ? 0 : slot + 1;
    };
    int s = 0;
    for (; s + 1 < nst; s += 2) {
        stage(S0{}, s);
        stage(S1{}, s + 1);
    }
    if (s < nst) stage(S0{}, s);

    // ---- epilogue: round16(fl32(acc) * alpha).  Lane l holds columns 4 (l >> 4) .. + 3 of row (l & 15) of a block; rows go out whole, 16
    // bytes per lane, through a part of the ring (free once everybody is here).
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    wait_vmcnt_imm<0>();
    __builtin_amdgcn_s_barrier();
    char* const stg = smem + wave * STG;
    const float alpha = p.alpha;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const v4i v = acc[i][j];
            const uint32_t o01 = dequant_pair<BF16>(v[0], v[1], alpha, alpha, 0.0f, 0.0f, false, false, 0u, false);
            const uint32_t o23 = dequant_pair<BF16>(v[2], v[3], alpha, alpha, 0.0f, 0.0f, false, false, 0u, false);
            *(v2u*)(stg + (i * 16 + r16) * PITCH + j * 32 + g * 8) = v2u{o01, o23};
        }
    __builtin_amdgcn_wave_barrier();
    uint16_t* const C = (uint16_t*)p.C + (int64_t)batch * p.strideC;
    constexpr int CPR = 2 * NB;  // 16-byte pieces per row
#pragma unroll
    for (int it = 0; it < (16 * MB * CPR + 63) / 64; ++it) {
        const int idx = it * 64 + lane, r = idx / CPR, c = idx - r * CPR;
        const v4u val = *(const v4u*)(stg + (r < 16 * MB ? r : 0) * PITCH + c * 16);
        if (r < rows && n0 + c * 8 < p.N) __builtin_nontemporal_store(val, (v4u*)(C + (int64_t)(w0 + r) * p.N + n0 + c * 8));
    }
}

template <int NB> void launch(const GemmArgs& a, int mb, dim3 grid, bool bf16, hipStream_t st)
{
    if (mb == 1) {
        if (bf16) sq_launch((pv_kernel<true, NB, 1>), grid, dim3(256), 0, st, a);
        else sq_launch((pv_kernel<false, NB, 1>), grid, dim3(256), 0, st, a);
    } else if (mb == 4) {
        if constexpr (NB >= 7) {
            if (bf16) sq_launch((pv_kernel<true, NB, 4>), grid, dim3(256), 0, st, a);
            else sq_launch((pv_kernel<false, NB, 4>), grid, dim3(256), 0, st, a);
        }
    } else {
        if (bf16) sq_launch((pv_kernel<true, NB, 2>), grid, dim3(256), 0, st, a);
        else sq_launch((pv_kernel<false, NB, 2>), grid, dim3(256), 0, st, a);
    }
}

// Rows of a wave (16, 32 or 64; four waves a workgroup).  Workgroups of 128 rows where two of them per compute unit keep it busy, else of 64 (B is
// fetched twice as often then); short rows end before the second one pays.  us, 64 / 128 rows: 32 x 448 x 448 x 80 (128 workgroups of 128)
// 4.8 / 5.5, 96 x 448 x 448 x 112 9.3 / 9.9, 128 x 448 x 448 x 112 (512) 11.7 / 10.7, 128 x 1024 x 1024 x 96 41.9 / 38.3; 600 x 128 x 128 x 80
// 6.6 / 7.1, 1200 of them 12.0 / 11.1.  Nor where blocks of 128 leave a quarter more rows empty (462 x 135 x 5264 x 32 95 / 140).
// Seven or eight column blocks and longer rows: what a workgroup reads of B and of the LDS per product counts, and A and B of many columns are read
// by several.  Then 128 rows already where those of 64 need a second round (three a compute unit: 15 x 3708 x 7904 x 128 149 / 122), with several
// column tiles from more than one of 64 a compute unit on (7 x 709 x 2448 x 1536 39.8 / 32.8), though not where they are just over one of 128 (3 x 902
// x 3680 x 1408 30.9 / 36.0) nor on shorter rows.  256 rows (two a compute unit) where they come to one round, to two, or to so many that the last does
// not count (532 of them, 2 x 4798 x 3376 x 1792, 128 / 256 rows: 89.5 / 100): 64 / 128 / 256 rows 8192 x 8192 x 8192 1265 / 766 / 605, 512 x 4096 x 16384
// 94 / 62 / 49, 768 x 2048 x 2048 x 128 932 / 796 / 714, 32 x 8192 x 8192 x 128 579 / 474 / 424.  Over 680 shapes within 3 % of the best of the three, and
// 0.57 of a 256 x 128 tile with both operands in LDS (679, 51, 806, 458 us on those four); 14 shapes lose more than 2 % to that tile, all of rows of 2600
// and more in one or two rounds, the worst 15 % (6 x 3796 x 2944 x 240 40.7 / 46.7).
int rows_per_wave(int64_t batch, int64_t m, int64_t k, int nb, int64_t tiles_n)
{
    auto padded = [&](int64_t r) { return (m + r - 1) / r * r; };
    auto groups = [&](int64_t r) { return batch * (padded(r) / r) * tiles_n; };
    const int64_t g64 = groups(64), g128 = groups(128), g256 = groups(256);
    const bool several = tiles_n > 1;
    if (nb >= 7 && k >= 512) {
        const bool no_more = padded(256) == padded(128);
        if (no_more && g256 >= 192 && g256 <= 256) return 64;
        if (k >= 1024 && g256 >= (several ? 400 : 480) && g256 <= 512 && padded(256) * 8 <= padded(128) * 9) return 64;
        if (k >= 1024 && no_more && g256 >= 768) return 64;
    }
    if (k >= 512 && g128 < 512 && padded(128) * 8 <= padded(64) * 9) {
        if (nb >= 7 && g64 > 768) return 32;
        if (nb >= 7 && several && g64 > 320 && (g128 <= 256 || (g128 > 288 && k >= 2048))) return 32;
        if (nb < 7 && several && g128 > 384 && k >= 2048) return 32;
    }
    if (g128 < (k < 256 ? 1024 : 512)) return 16;
    return padded(128) * 4 > padded(64) * 5 && (nb < 7 || (!several && k >= 1024)) ? 16 : 32;
}

}  // namespace

// a: M, N (a multiple of 16), K (of 16), lda = K, batch strides, alpha.
void sq_pv_bmm_launch(GemmArgs a, int batch, bool bf16, hipStream_t st)
{
    const int blocks = a.N / 16;
    a.tiles_n = (blocks + 7) / 8;
    const int nb = (blocks + a.tiles_n - 1) / a.tiles_n;
    const int mb = rows_per_wave(batch, a.M, a.K, nb, a.tiles_n) / 16;
    // A launch holds 2^32 threads: rows beyond that in further launches.
    const int64_t most = ((int64_t)1 << 23) / a.tiles_n * (64 * mb);
    const int64_t rows = a.M;
    for (int64_t r = 0; r < rows; r += most) {
        const int64_t now = rows - r < most ? rows - r : most;
        a.M = (int)now;
        const dim3 grid((unsigned)((now + 64 * mb - 1) / (64 * mb) * a.tiles_n), (unsigned)batch);
        switch (nb) {
            case 1: launch<1>(a, mb, grid, bf16, st); break;
            case 2: launch<2>(a, mb, grid, bf16, st); break;
            case 3: launch<3>(a, mb, grid, bf16, st); break;
            case 4: launch<4>(a, mb, grid, bf16, st); break;
            case 5: launch<5>(a, mb, grid, bf16, st); break;
            case 6: launch<6>(a, mb, grid, bf16, st); break;
            case 7: launch<7>(a, mb, grid, bf16, st); break;
            default: launch<8>(a, mb, grid, bf16, st); break;
        }
        a.A += most * a.lda;
        a.C = (uint16_t*)a.C + most * a.N;
    }
}
