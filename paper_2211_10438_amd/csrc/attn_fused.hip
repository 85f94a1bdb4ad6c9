// Fused INT8 attention for gfx950: O = (P_q V_q) * alpha2 with P_q = round(127 * softmax16(S)), S = round16((Q_q K_q^T) * alpha1),
// in one kernel that never writes the score or probability tensors.
//
// The attention block of Sec. 4 runs both batched matmuls in INT8 and keeps the softmax in the 16-bit
// floating type; the unfused chain (sq_w8a8_bmm, sq_softmax_quant_p, sq_w8a8_bmm) moves the [s_q, s_k]
// tensors S (16-bit) and P_q (int8) through HBM twice each, 19 of the 20 GB it touches at 768 heads x 2048^2.
// This kernel keeps the same quantization points -- scores rounded to 16 bits before the softmax,
// probabilities rounded to 16 bits and then to codes with the fixed step 1/127 -- and recomputes Q K^T
// instead of storing it:
//   pass 1  over the key tiles: S tile by MFMA, running row maximum and sum of exponentials (online softmax);
//   pass 2  over the key tiles again: S tile by MFMA, p = e^(s - m) / l, p16, code = round(127 p16); the 16
//           codes a lane produces from one 32x32 accumulator block ARE its operand fragment of the P V
//           MFMA (second operand: row l & 31, contraction bytes 16 (l >> 5) ..), so P_q never leaves registers.
// One workgroup owns 128 query rows of one (batch, head): four waves of 32 rows, the Q operand fragments in
// registers for the whole kernel.  K tiles of 128 keys (pass 1) and K and V tiles of 64 (pass 2; 128 at head dimension 64) travel L2 -> LDS with
// global_load_lds, double buffered, one s_barrier per tile.  Because the Q K^T MFMA takes the K rows as first operand, an
// accumulator block is the transpose of its output block: a lane holds, for its row, the columns 8g + 4h + e of a 32-key
// block (h = l >> 5).  That fixes the order of the contraction bytes of the P V MFMA; the V operand is fetched
// in the same order with the LDS transpose read (ds_read_b64_tr_b8), whose eight source rows are named by the
// lanes and can therefore be any eight keys.
// What bounds it: vector-ALU issue.  Measured on loops of single instructions (cycles per instruction and SIMD, with 2 / 4
// waves on it): add, sub, mul 3.0 / 2.7, conversions, packed and three-operand forms 5.1 / 4.5, exp2 8.8 / 8.4; one wave
// alone issues one every 6.2 whatever it is; a 32x32x32 MFMA runs beside them and takes about 8 issue cycles of its 34.
// Hence three workgroups per compute unit instead of two -- tiles of 64 keys, one accumulator pair live at a time, a single copy
// of the P V products --, no conversion of the sums where that pays (BIAS), and little done for keys and rows that are not
// there (MASK).  (A shift fixed by the first tile instead of the running maximum, half an instruction per score less,
// gained 1 %: the sums' last bits, and with them some codes, would no longer be those of a running maximum.)  With two
// workgroups per unit / now, us, timed in turn: 288 heads x 1024^2 x 128 causal 139 / 104, unmasked 184 / 171; 768 x 2048^2 x 128
// causal 1066 / 930, unmasked 1768 / 1636; 288 x 1024^2 x 64 unmasked 132 / 126; 96 x 777 x 1040 x 64 64.5 / 61.
#include <type_traits>

#include "attn_args.h"
#include "sqmi_probe.h"

namespace {

constexpr int kIntMin = -2147483647 - 1;
constexpr int kBias = 0x3e22f983;
constexpr float kBiasF = __builtin_bit_cast(float, kBias);

// MASK: one instantiation each, so that the common case carries no mask tests (with them in one kernel the register allocation
// spilled):
//   kAll     every query sees every key, and the key count is a multiple of 128;
//   kTail    the same with any key count: on the last, partial tile the 16-key groups that are there (s_k % 16 == 0), all of them
//            in full;
//   kCausal  query i sees the keys j <= i + p.coff (coff = s_k - s_q: the last query sees every key).  A workgroup stops after the
//            last tile any of its rows sees; a wave runs the plain tile body on the tiles all its 32 rows see in full, and
//            nothing on the tiles past its rows.  On the one or two tiles in between it takes the 32-key blocks one by one:
//            those its rows see in full without a mask, those they see in part with an element-wise one, of the others no
//            more than the products (a whole-tile masked body cost 1.7 plain ones on every diagonal tile, of which a 32-row group
//            sees between one and four blocks).
// BIAS: see kBias below.
constexpr int kAll = 0, kTail = 1, kCausal = 2;
template <bool BF16, int HD, int MASK, bool CODES, bool BIAS>
__global__ __launch_bounds__(256, 3) void attn_i8_kernel(const AttnArgs p)
{
    constexpr bool CAUSAL = MASK == kCausal, TAIL = MASK == kTail;
    constexpr int TK1 = 128, TK = HD == 64 ? 128 : 64;  // keys per tile of pass 1 (K only) and pass 2 (K and V)
    constexpr int KB = TK / 32;           // 32-key blocks per tile of pass 2
    constexpr int TILE = TK * HD;         // bytes of a K or V tile of pass 2
    constexpr int PITCH = HD * 2 + 16;    // bytes per row of the output staging
    constexpr int SLOT = TILE > 32 * PITCH ? TILE : (32 * PITCH + 1023) / 1024 * 1024;  // LDS bytes per tile (or staging of a wave)
    constexpr int LPT = TILE / 1024 / 4;  // global->LDS loads per wave and tile
    constexpr int CH = HD / 16;           // 16-byte chunks per row
    constexpr int RPB = 1024 / HD;        // rows per 1 KB block
    constexpr int NKS = HD / 32;          // MFMA steps of Q K^T
    constexpr int NB = HD / 32;           // 32-column blocks of O
    static_assert(HD == 128 || HD == 64, "head dimension");
    static_assert(TK1 * HD <= 2 * SLOT, "a pass 1 tile fits the K and V slots of a stage");
    __shared__ __attribute__((aligned(1024))) char smem[4 * SLOT];  // stage s: K tile at slot 2s, V tile at slot 2s + 1

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r32 = lane & 31, h = lane >> 5;

    // Which row block.  Without the mask each XCD gets a contiguous range of the logical order, so that the row blocks of one head
    // (they share its K and V) run on one L2.  (32-bit: the grid has fewer than 2^31 workgroups, and a 64-bit division is a
    // hundred scalar instructions)
    AttnPlace at;
    if constexpr (CAUSAL) {
        at = attn_causal_place(blockIdx.x, (uint32_t)p.batch, (uint32_t)p.tiles_m, (uint32_t)p.chunk);
    } else {
        const uint32_t xcd = blockIdx.x & 7, j = blockIdx.x >> 3, tiles = (uint32_t)p.tiles_m;
        const uint32_t per = gridDim.x >> 3, r = gridDim.x & 7, pid = xcd * per + (xcd < r ? xcd : r) + j, head = pid / tiles;
        at = {head, (int)(pid - head * tiles)};
    }
    const int64_t batch = at.batch;
    const int mt = at.tile;
    // The four row groups of 32 rotate over the waves from workgroup to workgroup: on the diagonal tile the last group sees
    // four times the keys of the first, and wave w of every workgroup sits on the same SIMD.
    const int rg = (wave + (blockIdx.x >> 3)) & 3;
    {
        const int m0 = mt * 128;
        const int w0 = m0 + rg * 32;      // first row of this wave
        const bool idle = w0 >= p.s_q;    // no row at all: the wave only fetches tiles
        // Keys the first and the last row of this wave see, and the last valid row of the workgroup (no row: none).  A tile that
        // ends at vmin or before is seen in full, one that starts at vmax or later not at all.
        int vmin = p.s_k, vmax = p.s_k, seen = p.s_k;
        if constexpr (CAUSAL) {
            const int last_row = m0 + 127 < p.s_q ? m0 + 127 : p.s_q - 1;
            auto sees = [&](int row) { return (int64_t)row + p.coff + 1 < p.s_k ? row + p.coff + 1 : p.s_k; };
            seen = sees(last_row);
            vmin = sees(w0);
            vmax = sees(w0 + 31);
            vmax = vmax < seen ? vmax : seen;
        }
        if (idle) vmin = vmax = 0;
        const int nt1 = (seen + TK1 - 1) / TK1, nt = (seen + TK - 1) / TK;  // tiles of the two passes
        // key index of accumulator register 4 g + e of key block ks in tile j: TK j + 32 ks + 8 g + 4 h + e; it is visible
        // to this lane's row when 32 ks + 8 g + e <= rowlim - TK j
        const int rowlim = ((int64_t)w0 + r32 + p.coff < p.s_k - 1 ? w0 + r32 + p.coff : p.s_k - 1) - 4 * h;  // (kCausal)

        // ---- LDS images.  K tile: row n at n * HD, its 16-byte chunks XOR-permuted (position = chunk ^ swzK(n)) so
        // that the operand reads (32 rows, one chunk) spread over the banks.  V tile: row k at k * HD, position =
        // chunk ^ swzV(k), chosen so that the eight rows of one transpose read sit at eight different positions.
        auto swzK = [](int r) { return HD == 128 ? (r & 7) : (((r >> 1) & 3) ^ ((r >> 3) & 1)); };
        auto swzV = [](int k) { return HD == 128 ? ((k & 3) | (((k >> 3) & 1) << 2)) : (k & 3); };
        // Key rows past s_k (last, partial tile) re-read row s_k - 1: their scores are masked below and their V rows meet
        // codes that are zero.
        // Slot i of this wave fills rows (4 i + wave) RPB ..: the swizzles of a lane's rows are the same for every i.
        const int lrow0 = wave * RPB + lane / CH;
        const uint32_t cK = (uint32_t)(((lane % CH) ^ swzK(lrow0)) * 16), cV = (uint32_t)(((lane % CH) ^ swzV(lrow0)) * 16);
        static_assert(4 * RPB % 16 == 0, "swizzles repeat every 16 rows");
        const int8_t* Kb = p.K + batch * p.stride_k;
        const int8_t* Vb = p.V + batch * p.stride_v;
        // (uniform base, 32-bit lane offset: no vector instruction per load.  The offset is made opaque next to the load, or its
        // widening to 64 bits is hoisted out of the loop and the scalar-base form of the load is lost.)
        auto load_tile = [&](const int8_t* base, uint32_t c, int k0, char* dst, auto LOADS_) {  // rows k0 .. of K or V
            constexpr int LOADS = decltype(LOADS_)::value;
            const int8_t* src = base + (int64_t)k0 * HD;
            uint32_t o[LOADS];  // this lane's byte of the tile; rows past the last key (the last, partial tile) stay on it
#pragma unroll
            for (int i = 0; i < LOADS; ++i) o[i] = (uint32_t)((lrow0 + i * 4 * RPB) * HD);
            if (MASK != kAll && k0 + LOADS * 4 * RPB > p.s_k) {
                const uint32_t last = (uint32_t)((p.s_k - 1 - k0) * HD);  // >= 0: the tile has a key
#pragma unroll
                for (int i = 0; i < LOADS; ++i) o[i] = o[i] < last ? o[i] : last;
            }
#pragma unroll
            for (int i = 0; i < LOADS; ++i) {
                uint32_t ok = o[i] + c;
                asm volatile("" : "+v"(ok));
                __builtin_amdgcn_global_load_lds(GPTR(src + ok), LPTR(dst + (i * 4 + wave) * 1024), 16, 0, 0);
            }
        };
        auto issue_k1 = [&](int j, int stage) {  // pass 1's tile j
            load_tile(Kb, cK, j * TK1, smem + (2 * stage) * SLOT, std::integral_constant<int, TK1 * HD / 4096>{});
        };
        auto issue = [&](int j, int stage) {  // pass 2's tile j
            load_tile(Kb, cK, j * TK, smem + (2 * stage) * SLOT, std::integral_constant<int, LPT>{});
            load_tile(Vb, cV, j * TK, smem + (2 * stage + 1) * SLOT, std::integral_constant<int, LPT>{});
        };

        // ---- Q operand fragments (second MFMA operand): lane l feeds query row (l & 31) of this wave with the 16
        // bytes of chunk 2 ks + (l >> 5).  Rows past s_q repeat the last row; they are never stored.
        v4i fq[NKS];
        {
            int row = w0 + r32;
            row = row < p.s_q ? row : p.s_q - 1;
            const int8_t* qp = p.Q + (int64_t)batch * p.stride_q + (int64_t)row * HD;
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) fq[ks] = *(const v4i*)(qp + (2 * ks + h) * 16);
        }
        // K operand fragment (first operand) of key block jn, step ks: key row 32 jn + (l & 31), chunk 2 ks + (l >> 5)
        // (position of chunk 2 ks + h = (2 ks) ^ (h ^ swz), so step ks flips bits 5.. of the address of step 0)
        const int koff0 = r32 * HD + ((h ^ swzK(r32)) * 16);
        // V operand fragment (first operand of the P V MFMA) of key block ks, column block jn: column n = 32 jn + (l & 31),
        // contraction bytes in the order the codes have in the P fragment: byte 4g + e <-> key 32 ks + 8g + 4h + e.
        // Within 16 lanes, source lanes 2j and 2j + 1 of a transpose read name the two 8-byte halves of the 16 columns
        // of one key row, and lane i receives column i of the eight rows: rows j = 0..3 are keys 4h + j, rows 4..7 keys
        // 8 + 4h + (j - 4); the second read takes the keys 16 further on.
        int voff;
        {
            const int s = lane & 15, j = s >> 1, cb = (lane >> 4) & 1;
            const int key = 4 * h + (j & 3) + 8 * (j >> 2);
            voff = key * HD + ((cb ^ swzV(key)) * 16) + (s & 1) * 8;  // chunk 2 jn + cb: jn enters below (XOR on bits 1.., swzV < 8)
        }
        auto v_frag = [&](const char* vt, int ks, int jn) {
            // position of chunk (2 jn + cb) = (2 jn + cb) ^ swz = ((2 jn) ^ (cb ^ swz)) as 2 jn has bit 0 clear
            const int a = (voff ^ ((2 * jn) << 4)) + ks * 32 * HD;
            const v2i lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((__attribute__((address_space(3))) v2i*)(vt + a));
            const v2i hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32((__attribute__((address_space(3))) v2i*)(vt + a + 16 * HD));
            return v4i{lo.x, lo.y, hi.x, hi.y};
        };

        // BIAS: the sums start at the bit pattern of kBias instead of at zero: read as a float, kBias + sum is the number
        // kBiasF + sum * 2^-26 exactly (|sum| <= 128^3 < 2292099, the distance of the pattern from the next power of two
        // below it), so one subtraction of kBiasF, exact too, replaces the conversion to float (a subtraction issues in half
        // the time of a conversion here).  The factor 2^26 is in alpha1.
        v16i bias;
#pragma unroll
        for (int v = 0; v < 16; ++v) bias[v] = BIAS ? kBias : 0;
        // S tile = Q K^T for the 128 keys of a stage: acc[jn] is the transposed 32x32 block of key block jn
        // (blocks from nvis on are left out)
        auto scores = [&](const char* kt, auto& acc, int nvis) {
            constexpr int N = sizeof(acc) / sizeof(v16i);
#pragma unroll
            for (int jn = 0; jn < N; ++jn) {
                if (jn >= nvis) break;
                acc[jn] = __builtin_amdgcn_mfma_i32_32x32x32_i8(*(const v4i*)(kt + jn * 32 * HD + koff0), fq[0], bias, 0, 0, 0);
            }
#pragma unroll
            for (int ks = 1; ks < NKS; ++ks)
#pragma unroll
                for (int jn = 0; jn < N; ++jn) {
                    if (jn >= nvis) break;
                    acc[jn] = __builtin_amdgcn_mfma_i32_32x32x32_i8(*(const v4i*)(kt + jn * 32 * HD + (koff0 ^ (ks << 5))), fq[ks], acc[jn], 0, 0, 0);
                }
        };
        // scores of two accumulators as the 16-bit tensor elements they stand for, widened again: round16(fl32(acc * alpha1)),
        // one narrowing instruction for the pair
        const float alpha1 = p.alpha1;  // BIAS: times 2^26
        auto s16f2 = [&](int a0, int a1, float& s0, float& s1) {
            auto sum = [](int a) { return BIAS ? __builtin_bit_cast(float, a) - kBiasF : (float)a; };
            const uint32_t h = store16x2_bits<BF16>(sum(a0) * alpha1, sum(a1) * alpha1);
            s0 = load16_bits<BF16>(h);
            s1 = load16_bits<BF16>(h >> 16);
        };
        // (Both passes must round the scores the same way: where one key dominates a row, l is 1 up to rounding, and a
        // score that came out one 16-bit ulp lower in pass 1 than in pass 2 would give that key a probability above 1.
        // A single-rounding v_fma_mixlo_f16 in pass 1 was tried for its one issue slot and did exactly that.)

        // ---- pass 1, tiles of 128 keys whatever pass 2's are (it needs no V and holds no output sums): row maximum m and
        // l = sum e^(s - m), online.  The maximum is taken on the integer accumulators (s is monotone in acc: alpha1 > 0).  A
        // row's scores are split between lanes r and r + 32.
        float m_run = -__builtin_inff(), l_run = 0.0f;
        using Plain = std::false_type;
        using Masked = std::true_type;
        // PART: a tile this wave's rows see in part: in units of 16 (kTail) or 32 (kCausal) keys, those below nfull in full, those
        // below nvis in part (keys up to lim), the others not at all; with kTail nfull = nvis
        constexpr int UNIT = TAIL ? 8 : 16;  // registers of a unit
        auto pass1_tile = [&](const char* kt, auto PART_, int lim, int nfull, int nvis) {
            constexpr bool PART = decltype(PART_)::value;
            v16i acc[4];
            scores(kt, acc, 4);  // (hidden blocks too: with the loads of the operands under a condition each MFMA waits for its own)
            int imax = kIntMin;
#pragma unroll
            for (int u = 0; u < 64 / UNIT; ++u) {
                if (PART && u >= nvis) break;
                const int jn = u * UNIT / 16, r0 = u * UNIT % 16;
                if (PART && CAUSAL && u >= nfull) {
#pragma unroll
                    for (int r = r0; r < r0 + UNIT; ++r) {  // register 4 g + e
                        const int a = 32 * jn + 8 * (r >> 2) + (r & 3) <= lim ? acc[jn][r] : kIntMin;
                        imax = a > imax ? a : imax;
                    }
                } else {
#pragma unroll
                    for (int r = r0; r < r0 + UNIT; ++r) imax = acc[jn][r] > imax ? acc[jn][r] : imax;
                }
            }
            const int other = __shfl_xor(imax, 32, 64);
            imax = other > imax ? other : imax;
            float s0, s1;
            s16f2(imax, imax, s0, s1);
            const float m_new = PART && CAUSAL && imax == kIntMin ? m_run : __builtin_fmaxf(m_run, s0);  // (a row may see nothing of a later tile)
            l_run *= __builtin_amdgcn_exp2f((m_run - m_new) * kLog2e);
            m_run = m_new;
            const float nm = -m_new * kLog2e;
            float part = 0.0f;
#pragma unroll
            for (int u = 0; u < 64 / UNIT; ++u) {
                if (PART && u >= nvis) break;
                const int jn = u * UNIT / 16, r0 = u * UNIT % 16;
                auto add = [&](auto EM_) {
                    constexpr bool EM = decltype(EM_)::value;
#pragma unroll
                    for (int r = r0; r < r0 + UNIT; r += 2) {
                        s16f2(acc[jn][r], acc[jn][r + 1], s0, s1);
                        const float e0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s0, kLog2e, nm));
                        const float e1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s1, kLog2e, nm));
                        const int idx = 32 * jn + 8 * (r >> 2) + (r & 3);
                        // (a hidden key's exponential may be anything, even infinite: it is dropped, not multiplied away)
                        part += (!EM || idx <= lim) ? e0 : 0.0f;
                        part += (!EM || idx + 1 <= lim) ? e1 : 0.0f;
                    }
                };
                if constexpr (PART && CAUSAL) {
                    if (u >= nfull) add(Masked{});
                    else add(Plain{});
                } else {
                    add(Plain{});
                }
            }
            l_run += part;
        };
        // 32-key blocks from key k0 on: seen in full by this wave's first row, and at all by its last
        auto n_full = [&](int k0) { return (vmin - k0) >> 5; };
        auto n_vis = [&](int k0, int most) { const int n = (vmax - k0 + 31) >> 5; return n < most ? n : most; };
        issue_k1(0, 0);
        for (int j = 0; j < nt1; ++j) {
            wait_vmcnt_imm<0>();           // this wave's part of tile j has landed
            __builtin_amdgcn_s_barrier();  // ... everybody's has, and everybody is done with tile j - 1
            // (behind the last tile the first one of pass 2, so that its latency is not exposed between the passes)
            if (j + 1 < nt1) issue_k1(j + 1, (j + 1) & 1);
            else issue(0, (j + 1) & 1);
            const char* kt1 = smem + (2 * (j & 1)) * SLOT;
            const int k0 = j * TK1;
            if (k0 + TK1 <= vmin) pass1_tile(kt1, Plain{}, 0, 8, 8);
            else if (CAUSAL && k0 < vmax) pass1_tile(kt1, Masked{}, rowlim - k0, n_full(k0), n_vis(k0, 4));
            else if (TAIL && k0 < vmax) pass1_tile(kt1, Masked{}, 0, (vmax - k0) >> 4, (vmax - k0) >> 4);
        }
        // p = e^(s - m) / l = 2^(s log2(e) - (m log2(e) + log2(l))): the division is folded into the exponent
        const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
        const float nm = -m_run * kLog2e - __builtin_amdgcn_logf(l_tot);

        // ---- pass 2: codes and P V.
        v16i acc_o[NB];
#pragma unroll
        for (int jn = 0; jn < NB; ++jn)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc_o[jn][v] = 0;
        int8_t* Prow = nullptr;
        if constexpr (CODES) {
            const int row = w0 + r32;
            if (row < p.s_q) Prow = p.P + ((int64_t)batch * p.s_q + row) * (int64_t)p.s_k + 4 * h;
        }
        // Tile j, its blocks below nvis; partial tiles drop the codes of the keys past lim = rowlim - TK j.  (One piece of code
        // for both: with a second copy of the P V products the accumulators are kept twice.)
        auto pass2_tile = [&](const char* kt, int j, bool partial, int lim, int nvis) {
            const char* vt = kt + SLOT;
            v16i acc[KB];
            scores(kt, acc, nvis);
#pragma unroll
            for (int ks = 0; ks < KB; ++ks) {
                if (MASK != kAll && ks >= nvis) break;
                v4i fp;  // the 16 codes of this lane: word g holds columns 8g + 4h + 0..3
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    if (TAIL && g == 2 && partial && 32 * ks + 16 >= lim) {  // (lim: keys of the tile) the block's second group is not there
                        fp[2] = fp[3] = 0;
                        break;
                    }
                    uint32_t ph[2];  // the probabilities of columns e = 0,1 and 2,3 as 16-bit pairs (the softmax output is a 16-bit tensor)
#pragma unroll
                    for (int e = 0; e < 4; e += 2) {
                        float s0, s1;
                        s16f2(acc[ks][4 * g + e], acc[ks][4 * g + e + 1], s0, s1);
                        ph[e >> 1] = store16x2_bits<BF16>(__builtin_amdgcn_exp2f(__builtin_fmaf(s0, kLog2e, nm)),
                                                          __builtin_amdgcn_exp2f(__builtin_fmaf(s1, kLog2e, nm)));
                    }
                    fp[g] = prob_codes4<BF16>(ph[0], ph[1]);
                }
                if (CAUSAL && partial) {
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const int n = lim - (32 * ks + 8 * g) + 1;  // visible keys of the four (or more)
                        const uint32_t m = n >= 4 ? 0xffffffffu : n <= 0 ? 0u : (1u << (8 * n)) - 1u;
                        fp[g] &= (int)m;
                    }
                }
                if (CODES && Prow) {
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        if (MASK == kAll || j * TK + ks * 32 + 8 * g + 4 * h < p.s_k) *(int*)(Prow + j * TK + ks * 32 + 8 * g) = fp[g];
                }
#pragma unroll
                for (int jn = 0; jn < NB; ++jn)
                    acc_o[jn] = __builtin_amdgcn_mfma_i32_32x32x32_i8(v_frag(vt, ks, jn), fp, acc_o[jn], 0, 0, 0);
            }
        };
        for (int j = 0; j < nt; ++j) {
            const int stage = (nt1 + j) & 1;
            wait_vmcnt_imm<0>();
            __builtin_amdgcn_s_barrier();
            if (j + 1 < nt) issue(j + 1, stage ^ 1);
            const char* kt2 = smem + (2 * stage) * SLOT;
            const int k0 = j * TK;
            if (k0 < vmax) pass2_tile(kt2, j, k0 + TK > vmin, TAIL ? vmax - k0 : rowlim - k0, MASK != kAll ? n_vis(k0, KB) : KB);
        }
        if constexpr (CAUSAL && CODES) {
            // the codes of the blocks this wave skipped are 0
            if (Prow)
                for (int c = (vmax + 31) / 32 * 32; c + 4 * h < p.s_k; c += 8) *(int*)(Prow + c) = 0;  // (Prow already points at column 4 h)
        }

        // ---- epilogue: o = round16(fl32(acc * alpha2)).  Accumulator block jn is the transposed output block: lane l,
        // register v holds row (l & 31), column 32 jn + 8 (v / 4) + 4 (l >> 5) + (v & 3).  Each wave stages its 32 rows in
        // its own part of the (now free) tile buffers and writes whole rows in 16-byte pieces.
        __syncthreads();
        char* stg = smem + wave * SLOT;
        const float alpha2 = p.alpha2;
#pragma unroll
        for (int jn = 0; jn < NB; ++jn)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const uint32_t o01 = dequant_pair<BF16>(acc_o[jn][4 * g], acc_o[jn][4 * g + 1], alpha2, alpha2, 0.0f, 0.0f, false, false, 0u, false);
                const uint32_t o23 = dequant_pair<BF16>(acc_o[jn][4 * g + 2], acc_o[jn][4 * g + 3], alpha2, alpha2, 0.0f, 0.0f, false, false, 0u, false);
                *(v2u*)(stg + r32 * PITCH + (32 * jn + 8 * g + 4 * h) * 2) = v2u{o01, o23};
            }
        __builtin_amdgcn_wave_barrier();
        uint16_t* Ob = (uint16_t*)p.O + (int64_t)batch * p.stride_o;
        constexpr int CPR = HD / 8;  // 16-byte pieces per row
#pragma unroll
        for (int it = 0; it < 32 * CPR / 64; ++it) {
            const int idx = it * 64 + lane, r = idx / CPR, c = idx - r * CPR;
            const int row = w0 + r;
            const v4u val = *(const v4u*)(stg + r * PITCH + c * 16);
            if (row < p.s_q) __builtin_nontemporal_store(val, (v4u*)(Ob + (int64_t)row * HD + c * 8));
        }
    }
}

}  // namespace

// Causal form: how many of its whole heads (every eighth) an XCD works on at a time.  Longest-first pays the more the fewer row
// blocks there are, and the chunks should be equal: all heads at once up to 16 MB of K and V per XCD (288 x 1024^2 x 128: 107 us
// against 112 in chunks of 8; 96 x 2048^2 121 against 135).  Beyond that their K and V should stay in the 4 MB L2 (768 x
// 2048^2: 969 us in chunks of 4 MB, 1071 all at once).
static int attn_chunk(int64_t b, int64_t s_k, int64_t d)
{
    const int64_t heads = b / 8, bytes = 2 * s_k * d;
    if (heads == 0) return 1;
    if (heads * bytes <= (16 << 20)) return (int)heads;
    int64_t n = (heads * bytes + (4 << 20) - 1) / (4 << 20);
    if (n > heads) n = heads;
    return (int)((heads + n - 1) / n);
}

// form: 0 by sq_attn_few_eligible, 1 row blocks, 2 few queries
static sq_status attention(int form, const int8_t* q, const int8_t* k, const int8_t* v, float alpha1, float alpha2, void* o,
                           sq_dtype out, int64_t b, int64_t s_q, int64_t s_k, int64_t d, int64_t stride_q,
                           int64_t stride_k, int64_t stride_v, int64_t stride_o, int8_t* p_codes, void* stream, bool causal)
{
    if (!q || !k || !v || !o) return SQ_ERR_NULL;
    const int64_t lim = (int64_t)1 << 31;
    if (b <= 0 || s_q <= 0 || s_k <= 0 || d <= 0 || s_q >= lim || s_k >= lim) return SQ_ERR_SHAPE;
    if (causal && s_k < s_q) return SQ_ERR_SHAPE;  // the first queries would see no key at all
    const int64_t tiles_m = (s_q + 127) / 128;
    if (b * tiles_m >= lim) return SQ_ERR_SHAPE;
    if (stride_q < s_q * d || stride_k < s_k * d || stride_v < s_k * d || stride_o < s_q * d) return SQ_ERR_SHAPE;
    if (out != SQ_F16 && out != SQ_BF16) return SQ_ERR_UNSUPPORTED;
    if (d != 64 && d != 128) return SQ_ERR_UNSUPPORTED;
    if (s_k & 15) return SQ_ERR_ALIGN;
    if (!(alpha1 > 0.0f) || !(alpha1 < __builtin_inff()) || !(alpha2 == alpha2)) return SQ_ERR_UNSUPPORTED;
    if ((stride_q & 15) || (stride_k & 15) || (stride_v & 15) || (stride_o & 7) || !sq_aligned16(q) || !sq_aligned16(k) ||
        !sq_aligned16(v) || !sq_aligned16(o) || (p_codes && (reinterpret_cast<uintptr_t>(p_codes) & 3u)))
        return SQ_ERR_ALIGN;
    AttnArgs a{};
    a.Q = q; a.K = k; a.V = v; a.O = o; a.P = p_codes;
    a.s_q = (int)s_q; a.s_k = (int)s_k;
    a.tiles_m = (int)tiles_m;
    a.stride_q = stride_q; a.stride_k = stride_k; a.stride_v = stride_v; a.stride_o = stride_o;
    a.alpha1 = alpha1; a.alpha2 = alpha2;
    hipStream_t st = (hipStream_t)stream;
    if (form == 0) form = sq_attn_few_eligible(b, s_q, s_k, d, causal) ? 2 : 1;
    if (form == 2) {
        if (!sq_attn_few_possible(b, s_q, s_k)) return SQ_ERR_UNSUPPORTED;
        sq_attn_few_launch(a, b, d, out == SQ_BF16, causal, st);
        return sq_launch_status();
    }
    a.batch = (int)b;
    a.coff = (int)(s_k - s_q);  // (kCausal)
    a.chunk = attn_chunk(b, s_k, d);
    const dim3 grid((unsigned)(b * tiles_m)), block(256);
    // BIAS where vector issue bounds the kernel: with masks, and more than two workgroups for a compute unit.  A workgroup that
    // has its unit to itself waits for the longer start of each sum instead (us, without / with: 768 x 2048^2 x 128 causal 954 /
    // 931, 100 x 1900^2 x 128 causal 129 / 126, 96 x 777 x 1040 x 64 61.5 / 60.8; but 64 x 512^2 x 128 16.5 / 16.8, 288 x 1024^2 x
    // 64 125 / 129, 2 x 16384^2 x 128 causal 421 / 428).
    const int mask = causal ? kCausal : (s_k & 127) != 0 ? kTail : kAll;
    const bool bias = mask != kAll && !p_codes && b * tiles_m > 512;
    // The kernel's scores carry a factor 2^-26 then.  A factor beyond 2^101 makes every difference of two scores infinite for
    // the softmax, like 2^101 itself.
    if (bias) a.alpha1 = (alpha1 < 0x1p+101f ? alpha1 : 0x1p+101f) * 0x1p+26f;
#define SQ_ATTN_K(BF, HD, MASK, CODES, BIAS) sq_launch((attn_i8_kernel<BF, HD, MASK, CODES, BIAS>), grid, block, 0, st, a)
#define SQ_ATTN_M(BF, HD, MASK)                                  \
    do {                                                         \
        if (p_codes) SQ_ATTN_K(BF, HD, MASK, true, false);       \
        else if (bias) SQ_ATTN_K(BF, HD, MASK, false, true);     \
        else SQ_ATTN_K(BF, HD, MASK, false, false);              \
    } while (0)
#define SQ_ATTN(BF, HD)                                          \
    do {                                                         \
        if (mask == kCausal) SQ_ATTN_M(BF, HD, kCausal);         \
        else if (mask == kTail) SQ_ATTN_M(BF, HD, kTail);        \
        else if (p_codes) SQ_ATTN_K(BF, HD, kAll, true, false);  \
        else SQ_ATTN_K(BF, HD, kAll, false, false);              \
    } while (0)
    if (d == 128) {
        if (out == SQ_BF16) SQ_ATTN(true, 128); else SQ_ATTN(false, 128);
    } else {
        if (out == SQ_BF16) SQ_ATTN(true, 64); else SQ_ATTN(false, 64);
    }
#undef SQ_ATTN
#undef SQ_ATTN_M
#undef SQ_ATTN_K
    return sq_launch_status();
}

extern "C" sq_status sq_w8a8_attention(const int8_t* q, const int8_t* k, const int8_t* v, float alpha1, float alpha2, void* o,
                                       sq_dtype out, int64_t b, int64_t s_q, int64_t s_k, int64_t d, int64_t stride_q,
                                       int64_t stride_k, int64_t stride_v, int64_t stride_o, int8_t* p_codes, void* stream)
{
    return attention(0, q, k, v, alpha1, alpha2, o, out, b, s_q, s_k, d, stride_q, stride_k, stride_v, stride_o, p_codes, stream, false);
}

extern "C" sq_status sq_w8a8_attention_causal(const int8_t* q, const int8_t* k, const int8_t* v, float alpha1, float alpha2, void* o,
                                              sq_dtype out, int64_t b, int64_t s_q, int64_t s_k, int64_t d, int64_t stride_q,
                                              int64_t stride_k, int64_t stride_v, int64_t stride_o, int8_t* p_codes, void* stream)
{
    return attention(0, q, k, v, alpha1, alpha2, o, out, b, s_q, s_k, d, stride_q, stride_k, stride_v, stride_o, p_codes, stream, true);
}

extern "C" int sq_probe_attention_form(int64_t b, int64_t s_q, int64_t s_k, int64_t d, int causal)
{
    if (b <= 0 || s_q <= 0 || s_k <= 0 || (d != 64 && d != 128)) return 0;
    return sq_attn_few_eligible(b, s_q, s_k, d, causal != 0) ? 2 : 1;
}

extern "C" int sq_probe_attention_place(int64_t block, int64_t b, int64_t s_q, int64_t s_k, int64_t d, int64_t* head)
{
    const int64_t tiles = (s_q + 127) / 128;
    if (b <= 0 || s_q <= 0 || s_k <= 0 || d <= 0 || block < 0 || !head || b * tiles >= ((int64_t)1 << 31) || block >= b * tiles) return -1;
    const AttnPlace at = attn_causal_place((uint32_t)block, (uint32_t)b, (uint32_t)tiles, (uint32_t)attn_chunk(b, s_k, d));
    *head = at.batch;
    return at.tile;
}

extern "C" sq_status sq_probe_attention(int form, int causal, const int8_t* q, const int8_t* k, const int8_t* v, float alpha1,
                                        float alpha2, void* o, sq_dtype out, int64_t b, int64_t s_q, int64_t s_k, int64_t d,
                                        int64_t stride_q, int64_t stride_k, int64_t stride_v, int64_t stride_o, int8_t* p_codes,
                                        void* stream)
{
    if (form != 1 && form != 2) return SQ_ERR_UNSUPPORTED;
    return attention(form, q, k, v, alpha1, alpha2, o, out, b, s_q, s_k, d, stride_q, stride_k, stride_v, stride_o, p_codes, stream, causal != 0);
}
