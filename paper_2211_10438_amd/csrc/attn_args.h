// Argument block of the fused attention kernels (gfx950).
#pragma once
#include "gemm_args.h"

struct AttnArgs {
    const int8_t* Q;  // [b][s_q, d]
    const int8_t* K;  // [b][s_k, d]
    const int8_t* V;  // [b][s_k, d]
    void* O;          // [b][s_q, d] 16-bit
    int8_t* P;        // optional [b][s_q, s_k]: the probability codes, for inspection; or NULL
    int s_q, s_k, tiles_m;  // tiles_m: workgroups (row blocks) per batch entry
    int batch, chunk;       // batch entries, and how many of them an XCD works on at a time
    int coff;               // causal: query i sees the keys j <= i + coff
    int64_t stride_q, stride_k, stride_v, stride_o;  // batch strides in elements
    float alpha1, alpha2;
};

constexpr float kLog2e = 1.44269504088896340736f;

struct AttnPlace {
    int64_t batch;
    int tile;  // row block
};
// Causal row-block form: what workgroup `block` works on.  Block t of a head sees t + 1 of the key tiles (the last queries every
// key), and consecutive workgroup ids go round-robin to the 8 XCDs, there to the next of 32 compute units.
//  * Longest first: the workgroups that start last decide when the launch ends.
//  * Whole heads go to the XCDs as far as they divide (XCD x: the heads x, x + 8, ..., `chunk` of them at a time, so that their K
//    and V stay in its L2).  The one to seven heads left over are dealt block by block, or XCDs would idle (1 x 32768^2 x 128 with
//    its head on one XCD 2050 us, dealt 868): sorted in by length, eight ranks at a time; with several chunks they come first.
//  * The first three workgroups of a compute unit start together.  The second round over the units runs backwards, so that a long
//    block shares its unit with a short one (12 x 8192^2 x 128 334 us without, 251 with).
__host__ __device__ __forceinline__ AttnPlace attn_causal_place(uint32_t block, uint32_t batch, uint32_t tiles, uint32_t chunk)
{
    const uint32_t xcd = block & 7, whole = batch >> 3, rest = batch & 7;
    uint32_t j = block >> 3;
    if ((j >> 5) == 1) {
        const uint32_t n = (batch * tiles + 7 - xcd) >> 3, hi = n < 64 ? n : 64;  // n: workgroups of this XCD
        j = 32 + (hi - 1 - j);
    }
    auto left_over = [&](uint32_t f, uint32_t r) { return AttnPlace{(int64_t)whole * 8 + (f - r * rest), (int)(tiles - 1 - r)}; };
    if (rest && chunk >= whole) {
        // eight ranks at a time (fewer at the end): of each left over head one block per XCD.  Number i of them on this XCD comes
        // in front of the whole heads' blocks of its rank.
        const uint32_t q = j / batch, full = tiles >> 3, p = q < full ? q : full, rank0 = 8 * p, ranks = q < full ? 8 : tiles - rank0;
        j -= p * batch;
        const uint32_t mine = (rest * ranks + 7 - xcd) >> 3, inv = 65536 / rest + 1;  // f / rest = (f * inv) >> 16 for f < 64
        uint32_t before = 0;
        for (uint32_t i = 0; i < mine; ++i) {
            const uint32_t f = i * 8 + xcd, r = (f * inv) >> 16, at = i + whole * r;
            if (at == j) return left_over(rank0 * rest + f, rank0 + r);
            if (at < j) before = i + 1;
        }
        j -= before;
        const uint32_t r = j / whole;
        return {(int64_t)(j - r * whole) * 8 + xcd, (int)(tiles - 1 - rank0 - r)};
    }
    if (rest) {
        const uint32_t mine = (rest * tiles + 7 - xcd) >> 3;
        if (j < mine) return left_over(j * 8 + xcd, (j * 8 + xcd) / rest);
        j -= mine;
    }
    const uint32_t c = j / (chunk * tiles);
    j -= c * (chunk * tiles);
    const uint32_t left = whole - c * chunk, heads = left < chunk ? left : chunk, r = j / heads;
    return {(int64_t)(c * chunk + (j - r * heads)) * 8 + xcd, (int)(tiles - 1 - r)};
}

// The 4 probability codes of two pairs of 16-bit probabilities (columns 0,1 in ph01, 2,3 in ph23), one byte each:
// round(127 p16), exactly rounded.
template <bool BF16> SQ_DEVICE int prob_codes4(uint32_t ph01, uint32_t ph23)
{
    if constexpr (BF16) {
        // the product is exact in fp32, the add of 1.5 * 2^23 rounds it to nearest-even and leaves the code in the low
        // mantissa byte
        const uint32_t ph[2] = {ph01, ph23};
        uint32_t q[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            q[e] = __builtin_bit_cast(uint32_t, __builtin_fmaf(load16_bits<true>(ph[e >> 1] >> ((e & 1) * 16)), 127.0f, 12582912.0f));
        return (int)pack4_low_bytes(q[0], q[1], q[2], q[3]);
    } else {
        // the same in packed fp16, two codes per instruction: fma(p16, 127, 1024) is one rounding of the exact
        // 127 p16 + 1024 to a grid of spacing 1 (fp16 in [1024, 2048)), i.e. 1024 + round-half-even(127 p16), the
        // code in the low byte of each half; one byte permute gathers the four codes
        const sq_f16x2 k127 = {(_Float16)127.0f, (_Float16)127.0f}, k1024 = {(_Float16)1024.0f, (_Float16)1024.0f};
        const uint32_t c01 = __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(__builtin_bit_cast(sq_f16x2, ph01), k127, k1024));
        const uint32_t c23 = __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(__builtin_bit_cast(sq_f16x2, ph23), k127, k1024));
        return (int)__builtin_amdgcn_perm(c23, c01, 0x06040200u);
    }
}

// Few queries over many keys (attn_few.hip): whether its registers and grid take a call at all, and whether it is the faster form.
bool sq_attn_few_possible(int64_t batch, int64_t s_q, int64_t s_k);
bool sq_attn_few_eligible(int64_t batch, int64_t s_q, int64_t s_k, int64_t d, bool causal);
void sq_attn_few_launch(AttnArgs a, int64_t batch, int64_t d, bool bf16, bool causal, hipStream_t st);
