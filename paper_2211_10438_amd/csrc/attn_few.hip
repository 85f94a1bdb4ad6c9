// Fused INT8 attention for few queries (the generation stage), gfx950: the same quantization points as attn_fused.hip --
// scores rounded to 16 bits, probabilities rounded to 16 bits and then to codes with the fixed step 1/127 -- with the work
// split along the keys instead of along the query rows.
//
// With one query per head the layer is bound by reading K and V once (2 d s_k bytes per head).  The row-block kernel gives
// a workgroup 128 query rows, computes all of them whatever s_q is, reads K twice and walks along the keys one tile at a
// time: 139 us at 768 heads x 1 x 2048 x 128 where the bytes take 62 at 6.5 TB/s (this kernel 66).  Here a workgroup owns at most 16 query
// rows of a head and its NW waves deal the 128-key groups among themselves:
//   phase 1  a wave loads the K rows of its groups straight into registers (v_mfma_i32_16x16x64_i8 takes 16 rows x 64 bytes
//            as they lie in memory, the next 64 in flight), keeps the 16-bit scores of ALL its groups in registers (16 per
//            group and lane, two scores each) and leaves each group's row maxima in LDS;
//   sums     with the running maximum over the groups up to its own known, a wave sums the exponentials of each group; the
//            row statistics are then folded group after group.  Sums and folds run in the order, and with the running maxima,
//            of the row-block kernel, so that both kernels give the same codes bit for bit (the sum of a row depends on the
//            order in its last bits, and a code may hang on those);
//   phase 2  probabilities, codes and P V per 64 keys; V arrives by LDS-DMA in a patch of the wave's own, two deep (the
//            first two are in flight across the sums), and is read with the LDS transpose read; no workgroup barriers.
// The int32 sums of the waves meet in LDS at the end.  The scores of a lane are 4 neighbouring keys of one query, and its 16
// codes of 64 keys (bytes 4 b + v <-> key 16 b + 4 (lane >> 4) + v) are its operand fragment of the P V MFMA; V is fetched in
// that order.
#include "attn_args.h"

namespace {

constexpr float kNegInf = -__builtin_inff();

template <bool BF16, int HD, int NW, int G>
__global__ __launch_bounds__(NW * 64, 2) void attn_few_kernel(const AttnArgs p, const int causal)
{
    constexpr int NKS = HD / 64;           // MFMA steps of Q K^T
    constexpr int NB = HD / 16;            // 16-column blocks of O
    constexpr int TILE = 64 * HD;          // bytes of the V rows of 64 keys
    constexpr int LV = TILE / 1024;        // LDS-DMA loads per 64 keys
    constexpr int CH = HD / 16, RPB = 1024 / HD;  // 16-byte chunks per row, rows per 1 KB
    constexpr int OP = HD + 4;             // ints per row of the output staging
    static_assert(HD == 128 || HD == 64, "head dimension");
    static_assert(16 * OP * 4 <= 2 * TILE, "output staging fits a wave's V patch");
    __shared__ __attribute__((aligned(1024))) char smem[NW * 2 * TILE];
    __shared__ float gmax[G * NW][16];     // row maxima of a group
    __shared__ float gsum[G * NW][2][16];  // its sums of exponentials, for the keys with bit 2 clear and set

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r16 = lane & 15, g = lane >> 4;

    // Consecutive workgroup ids go round-robin to the 8 XCDs; each XCD gets a contiguous range of the logical order, so
    // that the row blocks of one head run on one L2.
    uint32_t pid;
    {
        const uint32_t j = blockIdx.x >> 3, per = gridDim.x >> 3, xcd = blockIdx.x & 7, r = gridDim.x & 7;
        pid = xcd * per + (xcd < r ? xcd : r) + j;
    }
    const uint32_t head = pid / (uint32_t)p.tiles_m;
    const int64_t batch = head;
    const int q0 = (int)(pid - head * (uint32_t)p.tiles_m) * 16;
    const int last_q = q0 + 15 < p.s_q ? q0 + 15 : p.s_q - 1;
    // keys 0 .. row + coff are visible to a row; n_keys: those the last row of this workgroup sees
    const int coff = causal ? p.s_k - p.s_q : p.s_k;
    const int n_keys = last_q + coff + 1 < p.s_k ? last_q + coff + 1 : p.s_k;
    const int groups = (n_keys + 127) >> 7;
    const int ng = groups > wave ? (groups - wave + NW - 1) / NW : 0;  // groups of this wave: wave, wave + NW, ...
    // Its keys in halves of 64: half hi is keys khalf(hi) .. + 63, hi = 2 (number of the group within the wave) + 0 / 1.  Past
    // the last one comes the last one again (loads that nobody uses keep the number in flight the same on every path).
    auto khalf = [&](int hi) { const int c = hi < 2 * ng ? hi : 2 * ng - 1; return ((c >> 1) * NW + wave) * 128 + (c & 1) * 64; };
    const int myrow = q0 + r16 < p.s_q ? q0 + r16 : p.s_q - 1;  // rows past s_q repeat the last one; never stored
    const int lim0 = (myrow + coff < p.s_k - 1 ? myrow + coff : p.s_k - 1) - 4 * g;  // key 4 g + x is visible when x <= lim0

    const int8_t* Kb = p.K + batch * p.stride_k;
    const int8_t* Vb = p.V + batch * p.stride_v;

    // ---- V patch of this wave: row k at k * HD, its chunks permuted (position = chunk ^ swz(k)) so that the 32 rows a
    // transpose read touches lie over all banks.
    auto swz = [](int k) { return HD == 128 ? (k >> 1) & 7 : (k >> 2) & 3; };
    char* patch = smem + wave * 2 * TILE;
    auto issue_v = [&](int hi, int stage) {
        const int k0 = khalf(hi);
#pragma unroll
        for (int i = 0; i < LV; ++i) {
            const int row = i * RPB + lane / CH, pos = lane % CH;
            int k = k0 + row;
            k = k < p.s_k ? k : p.s_k - 1;  // (their codes are zero)
            __builtin_amdgcn_global_load_lds(GPTR(Vb + (int64_t)k * HD + ((pos ^ swz(row)) * 16)), LPTR(patch + stage * TILE + i * 1024), 16, 0, 0);
        }
    };
    int voff;
    {
        // within 16 lanes, lanes 2 j and 2 j + 1 name the halves of a key's 16 columns and lane i receives column i of
        // the eight keys: j = 0..3 key 4 g + j, j = 4..7 key 16 + 4 g + j - 4; the second read takes the keys 32 further on
        const int j = r16 >> 1, key = 4 * g + (j & 3) + 16 * (j >> 2);
        voff = key * HD + swz(key) * 16 + (r16 & 1) * 8;
    }
    // Four column blocks' fragments.  (In asm, with their wait: the compiler answers the transpose-read builtin, of which it
    // does not know what it reads, with a wait for every LDS-DMA in flight, the next rows' too.)
    auto v_frags = [&](const char* vt, int jn, v4i(&f)[4]) {
        const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)vt;
        const uint32_t a0 = base + (uint32_t)(voff ^ (jn << 4)), a1 = base + (uint32_t)(voff ^ ((jn + 1) << 4)),
                       a2 = base + (uint32_t)(voff ^ ((jn + 2) << 4)), a3 = base + (uint32_t)(voff ^ ((jn + 3) << 4));
        v2i lo0, lo1, lo2, lo3, hi0, hi1, hi2, hi3;
        asm volatile("ds_read_b64_tr_b8 %0, %8\n\tds_read_b64_tr_b8 %1, %8 offset:%12\n\t"
                     "ds_read_b64_tr_b8 %2, %9\n\tds_read_b64_tr_b8 %3, %9 offset:%12\n\t"
                     "ds_read_b64_tr_b8 %4, %10\n\tds_read_b64_tr_b8 %5, %10 offset:%12\n\t"
                     "ds_read_b64_tr_b8 %6, %11\n\tds_read_b64_tr_b8 %7, %11 offset:%12\n\t"
                     "s_waitcnt lgkmcnt(0)"
                     : "=&v"(lo0), "=&v"(hi0), "=&v"(lo1), "=&v"(hi1), "=&v"(lo2), "=&v"(hi2), "=&v"(lo3), "=&v"(hi3)
                     : "v"(a0), "v"(a1), "v"(a2), "v"(a3), "n"(32 * HD)
                     : "memory");
        f[0] = v4i{lo0.x, lo0.y, hi0.x, hi0.y};
        f[1] = v4i{lo1.x, lo1.y, hi1.x, hi1.y};
        f[2] = v4i{lo2.x, lo2.y, hi2.x, hi2.y};
        f[3] = v4i{lo3.x, lo3.y, hi3.x, hi3.y};
    };

    // ---- phase 1
    v4i fq[NKS];
    {
        const int8_t* qp = p.Q + batch * p.stride_q + (int64_t)myrow * HD + g * 16;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) fq[ks] = *(const v4i*)(qp + ks * 64);
    }
    v4i kb[2][4][NKS];
    auto load_k = [&](v4i(&dst)[4][NKS], int hi) {
        const int k0 = khalf(hi);
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            int k = k0 + b * 16 + r16;
            k = k < p.s_k ? k : p.s_k - 1;
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) dst[b][ks] = *(const v4i*)(Kb + (int64_t)k * HD + ks * 64 + g * 16);
        }
    };
    uint32_t sc[2 * G][4][2];  // scores of half hi, block b: keys 16 b + 4 g + 0,1 and + 2,3 as 16-bit pairs
    const float alpha1 = p.alpha1;
    float mx = kNegInf;
    auto phase1 = [&](auto HI_, auto&& self) -> void {
        constexpr int hi = decltype(HI_)::value;
        if constexpr (hi + 1 < 2 * G) load_k(kb[(hi + 1) & 1], hi + 1);  // on every path, so that the wait for this half's rows leaves these in flight
        __builtin_amdgcn_sched_barrier(0);  // (left alone, the loads sink to their first use)
        const int lim = lim0 - khalf(hi);
        if constexpr ((hi & 1) == 0) mx = kNegInf;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            v4i acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(kb[hi & 1][b][0], fq[0], v4i{0, 0, 0, 0}, 0, 0, 0);
            if constexpr (NKS == 2) acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(kb[hi & 1][b][1], fq[1], acc, 0, 0, 0);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t pr = store16x2_bits<BF16>((float)acc[2 * h] * alpha1, (float)acc[2 * h + 1] * alpha1);
                sc[hi][b][h] = pr;
#pragma unroll
                for (int e = 0; e < 2; ++e) mx = __builtin_fmaxf(mx, 16 * b + 2 * h + e <= lim ? load16_bits<BF16>(pr >> (16 * e)) : kNegInf);
            }
        }
        if constexpr (hi & 1) {
            mx = __builtin_fmaxf(mx, __shfl_xor(mx, 16, 64));
            mx = __builtin_fmaxf(mx, __shfl_xor(mx, 32, 64));
            if (lane < 16) gmax[(hi >> 1) * NW + wave][lane] = mx;
        }
        if constexpr (hi + 1 < 2 * G) {
            if (hi + 1 < 2 * ng) self(std::integral_constant<int, hi + 1>{}, self);
        }
    };
    if (ng > 0) {
        load_k(kb[0], 0);
        phase1(std::integral_constant<int, 0>{}, phase1);
        issue_v(0, 0);
        issue_v(1, 1);
    }
    auto meet = [&] {  // (not __syncthreads: the first V rows stay in flight)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    meet();

    // ---- sums.  The keys of a row with bit 2 = h lie in lanes g = h and g = h + 2, four of a 16-key block in each.  Two groups
    // are summed together: a swap of lane halves gives the lower lanes both halves of the first group's exponentials and the
    // upper lanes both of the second's, and each adds its group's 64 in the order of the keys.
    {
        float m_cur = kNegInf;
        int done = 0;  // groups whose maxima m_cur covers
        auto running_max = [&](int t) {
            for (; done <= t; ++done) m_cur = __builtin_fmaxf(m_cur, gmax[done][r16]);
            return m_cur;
        };
        auto sums = [&](auto PI_, auto&& self) -> void {
            constexpr int ga = 2 * decltype(PI_)::value, gb = ga + 1;
            const int ta = ga * NW + wave, tb = gb * NW + wave;
            const float nma = -running_max(ta) * kLog2e;
            const bool two = gb < ng;
            const float nmb = two ? -running_max(tb) * kLog2e : 0.0f;
            const int la = lim0 - ta * 128, lb = two ? lim0 - tb * 128 : -1;  // (no second group: nothing of it is visible)
            float part = 0.0f;
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                float lo[4], up[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const uint32_t pa = sc[2 * ga + (b >> 2)][b & 3][v >> 1], pb = sc[2 * gb + (b >> 2)][b & 3][v >> 1];
                    float ea = __builtin_amdgcn_exp2f(__builtin_fmaf(load16_bits<BF16>(pa >> (16 * (v & 1))), kLog2e, nma));
                    float eb = __builtin_amdgcn_exp2f(__builtin_fmaf(load16_bits<BF16>(pb >> (16 * (v & 1))), kLog2e, nmb));
                    ea = 16 * b + v <= la ? ea : 0.0f;
                    eb = 16 * b + v <= lb ? eb : 0.0f;
                    const auto sw = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, ea), __builtin_bit_cast(uint32_t, eb), false, false);
                    const uint32_t s0 = sw[0], s1 = sw[1];  // copies: a vector element is no object to cast from
                    lo[v] = __builtin_bit_cast(float, s0);
                    up[v] = __builtin_bit_cast(float, s1);
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) part += lo[v];
#pragma unroll
                for (int v = 0; v < 4; ++v) part += up[v];
            }
            const int t = lane < 32 ? ta : tb;
            if (lane < 32 || two) gsum[t][g & 1][r16] = part;
            if constexpr (gb + 1 < G) {
                if (gb + 1 < ng) self(std::integral_constant<int, decltype(PI_)::value + 1>{}, self);
            }
        };
        if (ng > 0) sums(std::integral_constant<int, 0>{}, sums);
    }
    meet();
    float M = kNegInf, L = 0.0f;
    for (int t = 0; t < groups; ++t) {
        const float m_new = __builtin_fmaxf(M, gmax[t][r16]);
        L *= __builtin_amdgcn_exp2f((M - m_new) * kLog2e);
        M = m_new;
        L += gsum[t][g & 1][r16];
    }
    L = L + __shfl_xor(L, 16, 64);
    const float nm = -M * kLog2e - __builtin_amdgcn_logf(L);  // p = 2^(s log2(e) - (M log2(e) + log2(L)))

    // ---- phase 2
    v4i acc_o[NB];
#pragma unroll
    for (int jn = 0; jn < NB; ++jn) acc_o[jn] = v4i{0, 0, 0, 0};
    int8_t* Prow = nullptr;
    if (p.P && q0 + r16 < p.s_q) Prow = p.P + (batch * p.s_q + q0 + r16) * (int64_t)p.s_k + 4 * g;
    auto phase2 = [&](auto HI_, auto&& self) -> void {
        constexpr int hi = decltype(HI_)::value;
        const int k0 = khalf(hi), lim = lim0 - k0;
        v4i fp;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            uint32_t ph[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float pr[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    pr[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(load16_bits<BF16>(sc[hi][b][h] >> (16 * e)), kLog2e, nm));
                    pr[e] = 16 * b + 2 * h + e <= lim ? pr[e] : 0.0f;
                }
                ph[h] = store16x2_bits<BF16>(pr[0], pr[1]);
            }
            fp[b] = prob_codes4<BF16>(ph[0], ph[1]);
            if (Prow && k0 + 16 * b < p.s_k) *(int*)(Prow + k0 + 16 * b) = fp[b];
        }
        wait_vmcnt_imm<LV>();  // this half's V rows have landed; the next half's may be in flight
        const char* vt = patch + (hi & 1) * TILE;
#pragma unroll
        for (int jn = 0; jn < NB; jn += 4) {
            v4i f[4];
            v_frags(vt, jn, f);
            if (jn + 4 == NB) issue_v(hi + 2, hi & 1);  // the last reads are done: the half can be filled again
#pragma unroll
            for (int i = 0; i < 4; ++i) acc_o[jn + i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f[i], fp, acc_o[jn + i], 0, 0, 0);
        }
        if constexpr (hi + 1 < 2 * G) {
            if (hi + 1 < 2 * ng) self(std::integral_constant<int, hi + 1>{}, self);
        }
    };
    if (ng > 0) phase2(std::integral_constant<int, 0>{}, phase2);
    if (Prow)  // groups no row of this workgroup sees
        for (int c = (groups + wave) * 128; c < p.s_k; c += NW * 128)
#pragma unroll
            for (int b = 0; b < 8; ++b)
                if (c + 16 * b < p.s_k) *(int*)(Prow + c + 16 * b) = 0;

    // ---- the waves' sums meet: accumulator block jn, register v of lane l is query l & 15, column 16 jn + 4 (l >> 4) + v
    wait_vmcnt_imm<0>();  // the refills past the end have landed: the patch is free
    int* stg = (int*)patch;
#pragma unroll
    for (int jn = 0; jn < NB; ++jn) *(v4i*)(stg + r16 * OP + 16 * jn + 4 * g) = acc_o[jn];
    __syncthreads();
    const float alpha2 = p.alpha2;
    uint16_t* Ob = (uint16_t*)p.O + batch * p.stride_o + (int64_t)q0 * HD;
    const int items = (last_q - q0 + 1) * (HD / 4);
    for (int i = threadIdx.x; i < items; i += NW * 64) {
        const int r = i / (HD / 4), c = (i - r * (HD / 4)) * 4;
        v4i s = {0, 0, 0, 0};
#pragma unroll
        for (int w = 0; w < NW; ++w) s += *(const v4i*)((const int*)(smem + w * 2 * TILE) + r * OP + c);
        const uint32_t o01 = dequant_pair<BF16>(s[0], s[1], alpha2, alpha2, 0.0f, 0.0f, false, false, 0u, false);
        const uint32_t o23 = dequant_pair<BF16>(s[2], s[3], alpha2, alpha2, 0.0f, 0.0f, false, false, 0u, false);
        *(v2u*)(Ob + r * HD + c) = v2u{o01, o23};
    }
}

template <bool BF16, int HD, int NW> void launch_g(const AttnArgs& a, unsigned grid, bool causal, hipStream_t st)
{
    const int g = ((a.s_k + 127) / 128 + NW - 1) / NW;
#define SQ_FEW(G) sq_launch((attn_few_kernel<BF16, HD, NW, G>), dim3(grid), dim3(NW * 64), 0, st, a, causal ? 1 : 0)
    if (g <= 2) SQ_FEW(2);
    else if (g <= 4) SQ_FEW(4);
    else SQ_FEW(8);
#undef SQ_FEW
}

constexpr int kFewKeys = 8 * 8 * 128;  // what the registers of eight waves hold

// Eight waves per workgroup where there is at most one workgroup per compute unit, or where four waves' registers do not hold
// the scores (8 groups of 128 keys each); else four, two workgroups per compute unit, so that one loads while the other is at
// its meeting or its epilogue.
int few_waves(double workgroups, int64_t s_k) { return workgroups <= 256.0 || s_k > 4 * 8 * 128 ? 8 : 4; }

}  // namespace

bool sq_attn_few_possible(int64_t batch, int64_t s_q, int64_t s_k)
{
    return s_k <= kFewKeys && (double)batch * (double)((s_q + 15) / 16) < (1 << 22);  // (a grid stays below 2^32 threads)
}

// Which of the two forms, by a model of the time of both in microseconds: a launch takes what its longest workgroup takes, or, with
// more workgroups, what the whole work takes spread over the 256 compute units.  This form's 16-row blocks fill the chip early
// and finish early, but each reads K and V once more, out of L2; the row-block form computes 128 rows per workgroup whatever s_q
// is, and one, two and three workgroups on a compute unit take 1, 1.5 and 2.3 times as long.  Fitted to 1190 shapes of 1 to 900
// heads, 1 to 2048 queries and 16 to 12000 keys, both forms and the earlier row-block version timed in turn.  The choice costs
// 0.3 % against the better form on the mean; 41 shapes take the worse one by more than 3 %, three by more than 16 % (528 x 4 x 96 x
// 128, 450 x 21 x 640 x 128 and 39 x 179 x 320 x 128: 1.19 to 1.34); none is slower than the earlier version by more than 4 %.  The
// line, us, this form / row blocks: 768 x 1 x 2048 x 128 66 / 139, 13 x 320^2 x 64 7.7 / 10.4, 64 x 208 x 1040 x 64 22.3 / 24.6, but 123 x
// 208 x 1040 x 64 34 / 26, 51 x 208^2 x 128 13.9 / 10.1, 42 x 320^2 x 128 18.9 / 12.8.
bool sq_attn_few_eligible(int64_t batch, int64_t s_q, int64_t s_k, int64_t d, bool causal)
{
    if (!sq_attn_few_possible(batch, s_q, s_k)) return false;
    const double rows = (double)(s_q - 1), all = (double)s_k;
    auto larger = [](double a, double b) { return a > b ? a : b; };

    const double row_per_cu = (double)batch * (double)((s_q + 127) / 128) / 256.0;
    const double row_keys = causal ? all - 0.5 * rows : all;  // a query sees on average
    auto row_form = [&](double start, double diagonal, double tile_ends, double per_key, double two, double three) {
        const double crowd = row_per_cu <= 1.0 ? 1.0 : row_per_cu <= 2.0 ? two : row_per_cu <= 3.0 ? three : three / 3.0 * row_per_cu;
        return start + (causal ? diagonal : 0.0) + per_key * larger(all + tile_ends, (row_keys + tile_ends) * crowd);
    };
    const double row_us = d == 64 ? row_form(2.4, 0.9, 44.0, 0.021, 1.5, 2.4) : row_form(2.0, 1.0, 78.0, 0.0265, 1.4, 2.25);

    const double few_wg = (double)batch * (double)((s_q + 15) / 16), few_per_cu = few_wg / 256.0;
    const int64_t groups = (s_k + 127) / 128, waves = few_waves(few_wg, s_k), per_wave = (groups + waves - 1) / waves;
    const double few_keys = causal ? all - 0.4 * rows : all;  // (its long blocks do not start first)
    const bool many_keys = s_k > 4 * 8 * 128;  // one workgroup of eight waves on a compute unit at a time
    const double few_us = d == 64 ? larger(4.5 + 0.9 * (double)per_wave + 0.38 * (double)groups, 5.4 + (0.87 + (many_keys ? 0.004 : 0.003) * few_keys) * few_per_cu)
                                  : larger(5.6 + 0.9 * (double)groups, 5.4 + (2.1 + (many_keys ? 0.009 : 0.006) * few_keys) * few_per_cu);
    return few_us < 0.95 * row_us;
}

void sq_attn_few_launch(AttnArgs a, int64_t batch, int64_t d, bool bf16, bool causal, hipStream_t st)
{
    a.tiles_m = (a.s_q + 15) / 16;
    const unsigned grid = (unsigned)(batch * a.tiles_m);
    const bool eight = few_waves((double)grid, a.s_k) == 8;
#define SQ_FEW(BF, HD) do { if (eight) launch_g<BF, HD, 8>(a, grid, causal, st); else launch_g<BF, HD, 4>(a, grid, causal, st); } while (0)
    if (d == 128) {
        if (bf16) SQ_FEW(true, 128); else SQ_FEW(false, 128);
    } else {
        if (bf16) SQ_FEW(true, 64); else SQ_FEW(false, 64);
    }
#undef SQ_FEW
}
