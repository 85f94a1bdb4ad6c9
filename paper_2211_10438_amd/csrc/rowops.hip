// Row-wise 16-bit floating point operators that sit between the INT8 kernels (Sec. 4 keeps Softmax
// and LayerNorm in FP16) fused with the quantization that feeds the next INT8 kernel, gfx950:
//   * softmax over attention scores + quantization of P with the fixed step 1/127,
//   * LayerNorm with the smoothing factors folded into gamma/beta + per-token dynamic quantization.
// One row per wave or workgroup, held in registers: one HBM pass, 2 B in + 1 B out.
#include "common.h"

namespace {

template <bool BF16> SQ_DEVICE void unpack8r(const v4u raw, float (&f)[8])
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        f[2 * e] = load16_bits<BF16>(raw[e]);
        f[2 * e + 1] = load16_bits<BF16>(raw[e] >> 16);
    }
}

// e^x for x <= 0 through the hardware 2^x instruction (v_exp_f32): about 3 ulp of fp32 where the result
// matters (x > -6), far below the half-ulp of the 16-bit rounding that follows; results below 2^-126 come
// out as 0, which is what their codes are anyway.  The library routine costs ~20 instructions per call and
// made this pass ALU-bound.
// e^(z - m) with the subtraction folded into one fused multiply-add: 2^(z * log2(e) + nm), nm = -m * log2(e)
// rounded once per row.  Against (z - m) * log2(e) the argument differs by at most ~2 of its ulps (|argument| < 64),
// i.e. a relative 1e-5 in the result, far below the half-ulp of the 16-bit rounding that follows.
SQ_DEVICE float fast_exp_shifted(float z, float nm) { return __builtin_amdgcn_exp2f(__builtin_fmaf(z, 1.44269504088896340736f, nm)); }
// Code of a probability p16 in [0, 1] (already rounded to the 16-bit type): round(p16 * 127) needs no clamp, and
// p16 * 127 is exact in fp32 (11 x 7 significant bits), so the fused multiply-add with 1.5 * 2^23 rounds exactly
// once, to nearest-even, like the separate multiply and add of code_bits.
SQ_DEVICE uint32_t prob_code_bits(float p16) { return __builtin_bit_cast(uint32_t, __builtin_fmaf(p16, 127.0f, 12582912.0f)); }

// Over the 256 threads of a workgroup.
SQ_DEVICE float block_max_r(float v, float* red)
{
    v = wave_max(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return __builtin_fmaxf(__builtin_fmaxf(red[0], red[1]), __builtin_fmaxf(red[2], red[3]));
}
SQ_DEVICE float block_sum_r(float v, float* red)
{
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

SQ_DEVICE v2u pack8(const uint32_t (&q)[8])  // code_bits words -> 8 bytes
{
    return v2u{pack4_low_bytes(q[0], q[1], q[2], q[3]), pack4_low_bytes(q[4], q[5], q[6], q[7])};
}

template <bool BF16, int NV>
__global__ __launch_bounds__(256) void softmax_quant_kernel(const uint16_t* __restrict__ s, int cols, int8_t* __restrict__ pq)
{
    __shared__ float red[4];
    const int64_t row = blockIdx.x;
    const v4u* sr = (const v4u*)(s + row * (int64_t)cols);
    const int nvec = cols >> 3;
    float z[NV][8];
    float mx = -__builtin_inff();
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = threadIdx.x + i * 256;
        if (idx < nvec) {
            unpack8r<BF16>(__builtin_nontemporal_load(sr + idx), z[i]);
#pragma unroll
            for (int e = 0; e < 8; ++e) mx = __builtin_fmaxf(mx, z[i][e]);
        }
    }
    mx = block_max_r(mx, red);
    // a row of -inf only (fully masked) has no maximum to shift by: its exponentials are 0 and so are its codes
    const float nmx = mx == -__builtin_inff() ? 0.0f : -mx * 1.44269504088896340736f;
    float sum = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = threadIdx.x + i * 256;
        if (idx < nvec) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                z[i][e] = fast_exp_shifted(z[i][e], nmx);
                sum += z[i][e];
            }
        }
    }
    sum = block_sum_r(sum, red);
    const float inv = sum > 0.0f ? 1.0f / sum : 0.0f;
    v2u* out = (v2u*)(pq + row * (int64_t)cols);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = threadIdx.x + i * 256;
        if (idx < nvec) {
            uint32_t q[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                // probability rounded to the 16-bit type first (the softmax output is a 16-bit tensor)
                const float p16 = load16_bits<BF16>(store16_bits<BF16>(z[i][e] * inv));
                q[e] = prob_code_bits(p16);
            }
            __builtin_nontemporal_store(pack8(q), out + idx);
        }
    }
}

// One row per wave (rows up to 4096 scores): four rows per 256-thread workgroup, the reductions are
// cross-lane shuffles only (no barriers), and every lane keeps NV 16-byte loads in flight, which is what a
// pass bound by HBM latency x bandwidth needs (a 256-thread workgroup per 4 KB row had 16 bytes per lane).
template <bool BF16, int NV>
__global__ __launch_bounds__(256) void softmax_quant_wave_kernel(const uint16_t* __restrict__ s, int64_t rows, int cols,
                                                                int8_t* __restrict__ pq)
{
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const v4u* sr = (const v4u*)(s + row * (int64_t)cols);
    const int nvec = cols >> 3;
    float z[NV][8];
    float mx = -__builtin_inff();
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = lane + i * 64;
        if (idx < nvec) {
            unpack8r<BF16>(__builtin_nontemporal_load(sr + idx), z[i]);
#pragma unroll
            for (int e = 0; e < 8; ++e) mx = __builtin_fmaxf(mx, z[i][e]);
        }
    }
    mx = wave_max(mx);
    // a row of -inf only (fully masked) has no maximum to shift by: its exponentials are 0 and so are its codes
    const float nmx = mx == -__builtin_inff() ? 0.0f : -mx * 1.44269504088896340736f;
    float sum = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = lane + i * 64;
        if (idx < nvec) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                z[i][e] = fast_exp_shifted(z[i][e], nmx);
                sum += z[i][e];
            }
        }
    }
    sum = wave_sum(sum);
    const float inv = sum > 0.0f ? 1.0f / sum : 0.0f;
    v2u* out = (v2u*)(pq + row * (int64_t)cols);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = lane + i * 64;
        if (idx < nvec) {
            uint32_t q[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float p16 = load16_bits<BF16>(store16_bits<BF16>(z[i][e] * inv));
                q[e] = prob_code_bits(p16);
            }
            __builtin_nontemporal_store(pack8(q), out + idx);
        }
    }
}

// One row per workgroup, two-pass statistics over the whole row in registers.  The sums have one fixed order, whatever the
// launch: the row's 16-byte vectors are dealt to VT strands (vector v to strand v % VT, a strand adds its NV vectors'
// elements one after the other), 64 neighbouring strands meet in a butterfly, and these sums are added as (0 + 1) + (2 + 3),
// then + ((4 + 5) + (6 + 7)).  A thread carries ST of the strands: the codes do not depend on it.
//
// A row is bound by its latencies: the loads, then three exchanges between the waves (mean, variance, maximum).  So every load
// is unconditional (one under a condition is waited for before the next is issued), the butterflies are vector instructions,
// and an exchange has cells of its own and one barrier.  Only the last of a strand's vectors can lie past the end of the row: it
// re-reads the row's last one, adds nothing to the sums, and in the maximum is that vector once more.
//
// KEEP: the differences from the mean stay in registers for the last pass instead of being taken again from the values: fewer registers and
// instructions where rows queue for the chip, but for a row alone the subtractions no longer come in one burst ahead of the chain
// of squares.  us, without / with: 4 x 8192 4.97 / 5.06, 64 x 6144 4.36 / 4.43; 1400 x 8192 13.3 / 12.4, 1400 x 6144 10.4 / 10.0, 768 x 14336 10.6 / 10.3.
// (With four strands they cost a wave per SIMD, with two of 512 more than they save: 2560 x 16384 36.5 / 38.1.)
template <bool BF16, int VT, int NV, int ST, bool FULL, bool KEEP>
__global__ __launch_bounds__(VT / ST, KEEP && ST == 2 && NV == 4 ? 4 : 1) void ln_quant_kernel(const uint16_t* __restrict__ x, int c_i, const float* __restrict__ gamma_f,
                                                           const float* __restrict__ beta_f, float eps, float* __restrict__ scale,
                                                           int8_t* __restrict__ xq, bool tiled)
{
    constexpr int W = VT / 64;  // 64-strand groups
    __shared__ __attribute__((aligned(16))) float cells[3][W];
    const int64_t row = blockIdx.x;
    const v4u* xr = (const v4u*)(x + row * (int64_t)c_i);
    const int nvec = c_i >> 3, lane = threadIdx.x & 63;
    const int group = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * ST;  // first of this wave's groups
    int idx[ST][NV];
    bool in[ST], any[ST];  // the strand's last vector lies in the row; that of any of the wave's 64 does
    v4u raw[ST][NV];
#pragma unroll
    for (int s = 0; s < ST; ++s) {
        any[s] = FULL || (group + s) * 64 + (NV - 1) * VT < nvec;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            idx[s][i] = (group + s) * 64 + lane + i * VT;
            if (i == NV - 1) {
                in[s] = FULL || idx[s][i] < nvec;
                idx[s][i] = in[s] ? idx[s][i] : nvec - 1;
            }
            raw[s][i] = __builtin_nontemporal_load(xr + idx[s][i]);
        }
    }
    auto exchange = [&](const float (&v)[ST], float* cell, auto&& op) {
        if (lane == 0) {
#pragma unroll
            for (int s = 0; s < ST; ++s) cell[group + s] = v[s];
        }
        __syncthreads();
        float4 q = *(const float4*)cell;
        float r = op(op(q.x, q.y), op(q.z, q.w));
        if constexpr (W == 8) {
            q = *(const float4*)(cell + 4);
            r = op(r, op(op(q.x, q.y), op(q.z, q.w)));
        }
        return r;
    };
    auto add = [](float a, float b) { return a + b; };
    auto max = [](float a, float b) { return __builtin_fmaxf(a, b); };
    float f[ST][NV][8], part[ST];
#pragma unroll
    for (int s = 0; s < ST; ++s) {
        part[s] = 0.0f;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            if (i == NV - 1 && !any[s]) break;
            unpack8r<BF16>(raw[s][i], f[s][i]);
            float v = part[s];
#pragma unroll
            for (int e = 0; e < 8; ++e) v += f[s][i][e];
            part[s] = i < NV - 1 || in[s] ? v : part[s];
        }
        part[s] = wave_sum(part[s]);
    }
    const float mean = exchange(part, cells[0], add) / (float)c_i;
#pragma unroll
    for (int s = 0; s < ST; ++s) {
        part[s] = 0.0f;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            if (i == NV - 1 && !any[s]) break;
            float v = part[s];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float d = f[s][i][e] - mean;
                v += d * d;
                if constexpr (KEEP) f[s][i][e] = d;
            }
            part[s] = i < NV - 1 || in[s] ? v : part[s];
        }
        part[s] = wave_sum(part[s]);
    }
    const float var = exchange(part, cells[1], add) / (float)c_i;
    const float rstd = 1.0f / sqrtf(var + eps);
#pragma unroll
    for (int s = 0; s < ST; ++s) {
        part[s] = 0.0f;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const float4 g0 = *(const float4*)(gamma_f + idx[s][i] * 8), g1 = *(const float4*)(gamma_f + idx[s][i] * 8 + 4);
            const float4 b0 = *(const float4*)(beta_f + idx[s][i] * 8), b1 = *(const float4*)(beta_f + idx[s][i] * 8 + 4);
            const float g[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
            const float b[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
            if (i == NV - 1 && !any[s]) break;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                f[s][i][e] = (KEEP ? f[s][i][e] : f[s][i][e] - mean) * rstd * g[e] + b[e];
                part[s] = __builtin_fmaxf(part[s], __builtin_fabsf(f[s][i][e]));
            }
        }
        part[s] = wave_max(part[s]);
    }
    const float a = exchange(part, cells[2], max);
    const float r = a > 0.0f ? 127.0f / a : 0.0f;
    if (threadIdx.x == 0) scale[row] = a / 127.0f;
#pragma unroll
    for (int s = 0; s < ST; ++s)
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            if (i == NV - 1 && !any[s]) break;
            uint32_t codes[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) codes[e] = code_bits(f[s][i][e] * r);
            if (i < NV - 1 || in[s]) __builtin_nontemporal_store(pack8(codes), (v2u*)code_dst(xq, row, idx[s][i] * 8, c_i, tiled));
        }
}

// The same for many rows: a workgroup walks through them, the next one's loads under way from the moment the present one is unpacked, its
// share of gamma and beta in registers for good.  With a row per workgroup the loads were in flight for a third of a row's time, and
// eight bytes of gamma and beta per element came out of the L2 behind them.  Two workgroups of 512 threads or three of 256 per compute
// unit measure best, and what is left is vector issue (85 % of the time).  us, a row per workgroup / this, inputs from memory: 4096 x
// 9216 tiled 38.6 / 32.5, 2100 x 9216 20.7 / 18.4, 4096 x 12288 44.1 / 37.5, 4096 x 5120 20.1 / 17.5.  Not kept: three or four workgroups
// of 512 (33.4, 35.0), two strands per thread or four vectors per strand (spills), another order of the waves in every second
// workgroup, so that their last vectors fall on other SIMDs (36.1), one kernel for both (the compiler then schedules the loads and sums of
// a row alone in another order, 1024 x 12288 12.7 / 13.1).  The second launch bound holds the four waves per SIMD of those workgroups.
template <bool BF16, int VT>
__global__ __launch_bounds__(VT, 4) void ln_quant_walk_kernel(const uint16_t* __restrict__ x, int t, int c_i, const float* __restrict__ gamma_f,
                                                              const float* __restrict__ beta_f, float eps, float* __restrict__ scale,
                                                              int8_t* __restrict__ xq, bool tiled)
{
    constexpr int NV = 3, ST = 1;  // (the strands' loops as above, one each: without them the compiler forms the bounds anew for every row, 4096 x 9216 27.2 / 27.4 us)
    constexpr int W = VT / 64;  // 64-strand groups
    __shared__ __attribute__((aligned(16))) float cells[3][W];
    int row = blockIdx.x;
    const int nvec = c_i >> 3, lane = threadIdx.x & 63;
    const int group = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * ST;  // first of this wave's groups
    int idx[ST][NV];
    bool in[ST], any[ST];  // the strand's last vector lies in the row; that of any of the wave's 64 does
    v4u raw[ST][NV];
#pragma unroll
    for (int s = 0; s < ST; ++s) {
        any[s] = (group + s) * 64 + (NV - 1) * VT < nvec;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            idx[s][i] = (group + s) * 64 + lane + i * VT;
            if (i == NV - 1) {
                in[s] = idx[s][i] < nvec;
                idx[s][i] = in[s] ? idx[s][i] : nvec - 1;
            }
        }
    }
    auto load_row = [&](int r) {
        const v4u* xr = (const v4u*)(x + r * (int64_t)c_i);
#pragma unroll
        for (int s = 0; s < ST; ++s)
#pragma unroll
            for (int i = 0; i < NV; ++i) raw[s][i] = __builtin_nontemporal_load(xr + idx[s][i]);
    };
    load_row(row);
    float gam[ST][NV][8], bet[ST][NV][8];
    auto load_affine = [&](int s, int i, float (&g)[8], float (&b)[8]) {
        const float4 g0 = *(const float4*)(gamma_f + idx[s][i] * 8), g1 = *(const float4*)(gamma_f + idx[s][i] * 8 + 4);
        const float4 b0 = *(const float4*)(beta_f + idx[s][i] * 8), b1 = *(const float4*)(beta_f + idx[s][i] * 8 + 4);
        g[0] = g0.x; g[1] = g0.y; g[2] = g0.z; g[3] = g0.w; g[4] = g1.x; g[5] = g1.y; g[6] = g1.z; g[7] = g1.w;
        b[0] = b0.x; b[1] = b0.y; b[2] = b0.z; b[3] = b0.w; b[4] = b1.x; b[5] = b1.y; b[6] = b1.z; b[7] = b1.w;
    };
#pragma unroll
    for (int s = 0; s < ST; ++s)
#pragma unroll
        for (int i = 0; i < NV; ++i) load_affine(s, i, gam[s][i], bet[s][i]);
    auto exchange = [&](const float (&v)[ST], float* cell, auto&& op) {
        if (lane == 0) {
#pragma unroll
            for (int s = 0; s < ST; ++s) cell[group + s] = v[s];
        }
        __syncthreads();
        float4 q = *(const float4*)cell;
        float r = op(op(q.x, q.y), op(q.z, q.w));
        if constexpr (W == 8) {
            q = *(const float4*)(cell + 4);
            r = op(r, op(op(q.x, q.y), op(q.z, q.w)));
        }
        return r;
    };
    auto add = [](float a, float b) { return a + b; };
    auto max = [](float a, float b) { return __builtin_fmaxf(a, b); };
    for (;;) {
        float f[ST][NV][8], part[ST];
#pragma unroll
        for (int s = 0; s < ST; ++s) {
            part[s] = 0.0f;
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                if (i == NV - 1 && !any[s]) break;
                unpack8r<BF16>(raw[s][i], f[s][i]);
                float v = part[s];
#pragma unroll
                for (int e = 0; e < 8; ++e) v += f[s][i][e];
                part[s] = i < NV - 1 || in[s] ? v : part[s];
            }
            part[s] = wave_sum(part[s]);
        }
        const bool more = row < t - (int)gridDim.x;
        if (more) load_row(row + (int)gridDim.x);
        const float mean = exchange(part, cells[0], add) / (float)c_i;
#pragma unroll
        for (int s = 0; s < ST; ++s) {
            part[s] = 0.0f;
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                if (i == NV - 1 && !any[s]) break;
                float v = part[s];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float d = f[s][i][e] - mean;
                    v += d * d;
                    f[s][i][e] = d;
                }
                part[s] = i < NV - 1 || in[s] ? v : part[s];
            }
            part[s] = wave_sum(part[s]);
        }
        const float var = exchange(part, cells[1], add) / (float)c_i;
        const float rstd = 1.0f / sqrtf(var + eps);
#pragma unroll
        for (int s = 0; s < ST; ++s) {
            part[s] = 0.0f;
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                if (i == NV - 1 && !any[s]) break;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    f[s][i][e] = f[s][i][e] * rstd * gam[s][i][e] + bet[s][i][e];
                    part[s] = __builtin_fmaxf(part[s], __builtin_fabsf(f[s][i][e]));
                }
            }
            part[s] = wave_max(part[s]);
        }
        const float a = exchange(part, cells[2], max);
        const float r = a > 0.0f ? 127.0f / a : 0.0f;
        if (threadIdx.x == 0) scale[row] = a / 127.0f;
#pragma unroll
        for (int s = 0; s < ST; ++s)
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                if (i == NV - 1 && !any[s]) break;
                uint32_t codes[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) codes[e] = code_bits(f[s][i][e] * r);
                if (i < NV - 1 || in[s]) __builtin_nontemporal_store(pack8(codes), (v2u*)code_dst(xq, row, idx[s][i] * 8, c_i, tiled));
            }
        if (!more) break;
        row += (int)gridDim.x;
    }
}

// One row per wave (hidden sizes up to 2048, where it measures faster than a workgroup per row): the three
// reductions are cross-lane shuffles, no barriers, and a lane keeps NV 16-byte loads in flight.
template <bool BF16, int NV, bool KEEP>
__global__ __launch_bounds__(256) void ln_quant_wave_kernel(const uint16_t* __restrict__ x, int64_t t, int c_i,
                                                           const float* __restrict__ gamma_f, const float* __restrict__ beta_f,
                                                           float eps, float* __restrict__ scale, int8_t* __restrict__ xq, bool tiled)
{
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= t) return;
    const v4u* xr = (const v4u*)(x + row * (int64_t)c_i);
    const int nvec = c_i >> 3;
    float f[NV][8];
    float sum = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = lane + i * 64;
        if (idx < nvec) {
            unpack8r<BF16>(__builtin_nontemporal_load(xr + idx), f[i]);
#pragma unroll
            for (int e = 0; e < 8; ++e) sum += f[i][e];
        }
    }
    const float mean = wave_sum(sum) / (float)c_i;
    float sq = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = lane + i * 64;
        if (idx < nvec) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float d = f[i][e] - mean;
                sq += d * d;
                if constexpr (KEEP) f[i][e] = d;
            }
        }
    }
    const float var = wave_sum(sq) / (float)c_i;
    const float rstd = 1.0f / sqrtf(var + eps);
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = lane + i * 64;
        if (idx < nvec) {
            const float4 g0 = *(const float4*)(gamma_f + idx * 8), g1 = *(const float4*)(gamma_f + idx * 8 + 4);
            const float4 b0 = *(const float4*)(beta_f + idx * 8), b1 = *(const float4*)(beta_f + idx * 8 + 4);
            const float g[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
            const float b[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                f[i][e] = (KEEP ? f[i][e] : f[i][e] - mean) * rstd * g[e] + b[e];
                m = __builtin_fmaxf(m, __builtin_fabsf(f[i][e]));
            }
        }
    }
    const float a = wave_max(m);
    const float r = a > 0.0f ? 127.0f / a : 0.0f;
    if (lane == 0) scale[row] = a / 127.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = lane + i * 64;
        if (idx < nvec) {
            uint32_t q[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) q[e] = code_bits(f[i][e] * r);
            __builtin_nontemporal_store(pack8(q), (v2u*)code_dst(xq, row, idx * 8, c_i, tiled));
        }
    }
}

}  // namespace

extern "C" {

sq_status sq_softmax_quant_p(const void* s, sq_dtype dtype, int64_t rows, int64_t cols, int8_t* pq, void* stream)
{
    if (!s || !pq) return SQ_ERR_NULL;
    if (rows <= 0 || cols <= 0 || rows >= ((int64_t)1 << 31)) return SQ_ERR_SHAPE;
    if (dtype != SQ_F16 && dtype != SQ_BF16) return SQ_ERR_UNSUPPORTED;
    if (cols > 8 * 256 * 8) return SQ_ERR_UNSUPPORTED;  // rows up to 16384 scores
    if ((cols & 7) || !sq_aligned16(s) || !sq_aligned16(pq)) return SQ_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    const int nvec = (int)(cols >> 3);
    const uint16_t* sp = (const uint16_t*)s;
#define SQ_SM(BF, NV) sq_launch((softmax_quant_kernel<BF, NV>), dim3((unsigned)rows), dim3(256), 0, st, sp, (int)cols, pq)
#define SQ_SMW(BF, NV) sq_launch((softmax_quant_wave_kernel<BF, NV>), dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st, sp, rows, (int)cols, pq)
    if (dtype == SQ_BF16) {
        if (nvec <= 64) SQ_SMW(true, 1); else if (nvec <= 128) SQ_SMW(true, 2); else if (nvec <= 256) SQ_SMW(true, 4);
        else if (nvec <= 512) SQ_SMW(true, 8); else if (nvec <= 1024) SQ_SM(true, 4); else SQ_SM(true, 8);
    } else {
        if (nvec <= 64) SQ_SMW(false, 1); else if (nvec <= 128) SQ_SMW(false, 2); else if (nvec <= 256) SQ_SMW(false, 4);
        else if (nvec <= 512) SQ_SMW(false, 8); else if (nvec <= 1024) SQ_SM(false, 4); else SQ_SM(false, 8);
    }
#undef SQ_SM
#undef SQ_SMW
    return sq_launch_status();
}

sq_status sq_ln_quantize(const void* x, sq_dtype dtype, int64_t t, int64_t c_i, const float* gamma_f, const float* beta_f,
                         float eps, float* scale, int8_t* xq, sq_layout xq_layout, void* stream)
{
    if (!x || !gamma_f || !beta_f || !scale || !xq) return SQ_ERR_NULL;
    if (t <= 0 || c_i <= 0 || t >= ((int64_t)1 << 31)) return SQ_ERR_SHAPE;
    if (dtype != SQ_F16 && dtype != SQ_BF16) return SQ_ERR_UNSUPPORTED;
    if (c_i > 8 * 256 * 8) return SQ_ERR_UNSUPPORTED;  // hidden sizes up to 16384
    if (xq_layout != SQ_ROW_MAJOR && xq_layout != SQ_TILED) return SQ_ERR_UNSUPPORTED;
    if (xq_layout == SQ_TILED && (c_i & 63)) return SQ_ERR_ALIGN;
    const bool tiled = xq_layout == SQ_TILED;
    if ((c_i & 15) || !sq_aligned16(x) || !sq_aligned16(xq) || !sq_aligned16(gamma_f) || !sq_aligned16(beta_f))
        return SQ_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    const int nvec = (int)(c_i >> 3);
    const uint16_t* xp = (const uint16_t*)x;
    // Up to 2048 channels one row per wave; wider rows one per workgroup, with 1, 2 or 4 strands per thread (ST).  Short threads
    // have the shorter latency per row and win while all rows are in flight at once (us at 1 x 5120 with ST = 1 / 2 / 4: 3.7 /
    // 4.6 / 6.2, 1024 x 9216: 8.6 / 8.8 / 9.8).  Longer ones share the exchanges and take fewer registers for a row, so that
    // more rows fit a compute unit: with two vectors per strand 8 / 12 / 16, with three of 256 strands 8 / 8 / 12, of 512 strands
    // 4 / 4 / 6, with four 8 / 8 / 8 or 4 / 4 / 4.  The lines lie where the rows stop fitting (x 256 compute units), except that
    // between one and two rounds the form with the shortest tail wins (4096 x 4096 tiled 15.9 / 12.9 / 12.3, 2800 x 6144 17.4 /
    // 17.4 / 14.8, 1400 x 12288 17.5 / 17.8 / 15.0, 2048 x 8192 16.9 / 12.9 / 13.5, 4096 x 16384 56.9 / 54.2 / 56.2).  Against the
    // version with loads under a condition and two barriers an exchange: 4096 x 9216 tiled 37.9 -> 33.3 us, 1024 x 9216 11.7 ->
    // 8.7, 1 x 5120 4.4 -> 3.7.  Rows of three vectors per strand beyond one round of the four-strand form walk: of 512 strands
    // 1536 x 9216 13.1 without / 14.4 with, 1700 16.1 / 15.0; of 256 strands 3000 x 5120 13.4 / 14.7, 3600 19.6 / 16.9.  Differences kept (KEEP) beyond
    // two rows per compute unit (300 x 7680 6.01 / 6.08, 600 x 7680 7.04 / 7.02, 1400 12.8 / 12.3), a wave's rows beyond four per SIMD (2560 x 1296 6.35 / 6.40, 4096
    // 7.35 / 7.20, 5500 10.4 / 8.7; 2560 x 2048 7.50 / 7.56, 5500 14.0 / 12.2).
#define SQ_LNK(BF, VT, NV, ST, FULL, KEEP) sq_launch((ln_quant_kernel<BF, VT, NV, ST, FULL, KEEP>), dim3((unsigned)t), dim3(VT / ST), 0, st, xp, (int)c_i, gamma_f, beta_f, eps, scale, xq, tiled)
#define SQ_LNL(BF, VT, PER_CU) sq_launch((ln_quant_walk_kernel<BF, VT>), dim3(256 * PER_CU), dim3(VT), 0, st, xp, (int)t, (int)c_i, gamma_f, beta_f, eps, scale, xq, tiled)
#define SQ_LNW(BF, NV, KEEP) sq_launch((ln_quant_wave_kernel<BF, NV, KEEP>), dim3((unsigned)((t + 3) / 4)), dim3(256), 0, st, xp, t, (int)c_i, gamma_f, beta_f, eps, scale, xq, tiled)
#define SQ_LN1(BF, NV, FULL)                                                                                                  \
    do {                                                                                                                      \
        if (t <= 512) SQ_LNK(BF, 256, NV, 1, FULL, false);                                                                    \
        else SQ_LNK(BF, 256, NV, 1, FULL, true);                                                                              \
    } while (0)
#define SQ_LN2(BF, FULL)                                                                                                      \
    do {                                                                                                                      \
        if (t <= 2048) SQ_LN1(BF, 2, FULL);                                                                                   \
        else if (t <= 3072) SQ_LNK(BF, 256, 2, 2, FULL, true);                                                                \
        else SQ_LNK(BF, 256, 2, 4, FULL, false);                                                                              \
    } while (0)
#define SQ_LNA(BF)                                                                                                            \
    do {                                                                                                                      \
        if (nvec <= 128 && t <= 4096) SQ_LNW(BF, 2, false);                                                                   \
        else if (nvec <= 128) SQ_LNW(BF, 2, true);                                                                            \
        else if (nvec <= 256 && t <= 4096) SQ_LNW(BF, 4, false);                                                              \
        else if (nvec <= 256) SQ_LNW(BF, 4, true);                                                                            \
        else if (nvec < 512) SQ_LN2(BF, false);                                                                               \
        else if (nvec == 512) SQ_LN2(BF, true);                                                                               \
        else if (nvec <= 768) {                                                                                               \
            if (t > 3584) SQ_LNL(BF, 256, 3);                                                                                 \
            else if (t <= 1600 || t > 3072) SQ_LN1(BF, 3, false);                                                             \
            else if (t <= 2048) SQ_LNK(BF, 256, 3, 2, false, true);                                                           \
            else SQ_LNK(BF, 256, 3, 4, false, false);                                                                         \
        } else if (nvec <= 1024) {                                                                                            \
            if (t <= 1400 || (t > 2048 && t <= 2560)) SQ_LN1(BF, 4, false);                                                   \
            else if (t <= 3072) SQ_LNK(BF, 256, 4, 2, false, true);                                                           \
            else SQ_LNK(BF, 256, 4, 4, false, false);                                                                         \
        } else if (nvec <= 1536) {                                                                                            \
            if (t > 1536) SQ_LNL(BF, 512, 2);                                                                                 \
            else if (t <= 1024) SQ_LNK(BF, 512, 3, 1, false, false);                                                          \
            else SQ_LNK(BF, 512, 3, 4, false, false);                                                                         \
        } else if (t <= 768) SQ_LNK(BF, 512, 4, 1, false, true);                                                              \
        else SQ_LNK(BF, 512, 4, 2, false, false);                                                                             \
    } while (0)
    if (dtype == SQ_BF16) SQ_LNA(true);
    else SQ_LNA(false);
#undef SQ_LNK
#undef SQ_LNL
#undef SQ_LNW
#undef SQ_LN1
#undef SQ_LN2
#undef SQ_LNA
    return sq_launch_status();
}

}  // extern "C"
