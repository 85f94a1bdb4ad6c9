// Row-wise 16-bit floating point operators that sit between the INT8 kernels (Sec. 4 keeps Softmax
// and LayerNorm in FP16) fused with the quantization that feeds the next INT8 kernel, gfx950:
//   * softmax over attention scores + quantization of P with the fixed step 1/127,
//   * LayerNorm with the smoothing factors folded into gamma/beta + per-token dynamic quantization.
// One row per 256-thread workgroup, the row held in registers: one HBM pass, 2 B in + 1 B out.
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

template <int NT = 256> SQ_DEVICE float block_max_r(float v, float* red)
{
    v = wave_max(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    float m = __builtin_fmaxf(__builtin_fmaxf(red[0], red[1]), __builtin_fmaxf(red[2], red[3]));
#pragma unroll
    for (int w = 4; w < NT / 64; w += 4)
        m = __builtin_fmaxf(m, __builtin_fmaxf(__builtin_fmaxf(red[w], red[w + 1]), __builtin_fmaxf(red[w + 2], red[w + 3])));
    return m;
}
template <int NT = 256> SQ_DEVICE float block_sum_r(float v, float* red)
{
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    float t = (red[0] + red[1]) + (red[2] + red[3]);
#pragma unroll
    for (int w = 4; w < NT / 64; w += 4) t += (red[w] + red[w + 1]) + (red[w + 2] + red[w + 3]);
    return t;
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

// One row per workgroup of up to 512 threads, NV 16-byte vectors per thread, as many threads as that takes.  A wave forms the
// mean and the sum of squared deviations of its own part of the row (two-pass, in registers), and the parts are combined
// by the parallel-variance formula, mean = sum S_w / n, M2 = sum (M2_w + n_w (mean_w - mean)^2): two workgroup-wide exchanges
// per row, statistics and maximum, instead of three, and one barrier each.
template <bool BF16, int NV>
__global__ __launch_bounds__(512) void ln_quant_kernel(const uint16_t* __restrict__ x, int c_i, const float* __restrict__ gamma_f,
                                                       const float* __restrict__ beta_f, float eps, float* __restrict__ scale,
                                                       int8_t* __restrict__ xq, bool tiled)
{
    __shared__ float4 part_of[8];  // sum, mean, sum of squared deviations and number of elements of a wave
    __shared__ float wmax[8];
    const int64_t row = blockIdx.x;
    const v4u* xr = (const v4u*)(x + row * (int64_t)c_i);
    const int nvec = c_i >> 3, nt = blockDim.x, waves = nt >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Vectors past the end of the row re-read its last one (every load unconditional: a load under a condition is waited for
    // before the next one is issued, which made a row of NV vectors per thread NV memory latencies long, for x as for
    // gamma and beta); they take no part in the sums, and in the maximum and the codes they are that vector once more.
    int idx[NV];
    v4u raw[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        idx[i] = threadIdx.x + i * nt;
        idx[i] = idx[i] < nvec ? idx[i] : nvec - 1;
        raw[i] = __builtin_nontemporal_load(xr + idx[i]);
    }
    float f[NV][8];
    float sum = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        unpack8r<BF16>(raw[i], f[i]);
        float part = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) part += f[i][e];
        sum += (int)threadIdx.x + i * nt < nvec ? part : 0.0f;
    }
    // elements of this wave: its 64 lanes hold vectors wave * 64 + i * nt + 0 .. 63
    int n = 0;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int left = nvec - (wave * 64 + i * nt);
        n += left <= 0 ? 0 : left < 64 ? left : 64;
    }
    const float wn = (float)(8 * n);  // at least 8: the launch has no wave without a vector
    sum = wave_sum(sum);
    const float wmean = sum / wn;
    float sq = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        float part = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float d = f[i][e] - wmean;
            part = __builtin_fmaf(d, d, part);
        }
        sq += (int)threadIdx.x + i * nt < nvec ? part : 0.0f;
    }
    sq = wave_sum(sq);
    if ((threadIdx.x & 63) == 0) {
        part_of[wave] = float4{sum, wmean, sq, wn};
    }
    __syncthreads();
    // every group of eight lanes holds the waves' parts, one per lane, and reduces them
    auto sum8 = [](float v) { v += lane_xor<4>(v); v += lane_xor<2>(v); return v + lane_xor<1>(v); };
    const int w8 = threadIdx.x & 7;
    const float4 q = w8 < waves ? part_of[w8] : float4{0.0f, 0.0f, 0.0f, 0.0f};
    const float mean = sum8(q.x) / (float)c_i;
    const float d = q.y - mean;
    const float m2 = sum8(q.z + q.w * (d * d));
    const float rstd = 1.0f / sqrtf(m2 / (float)c_i + eps);
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const float4 g0 = *(const float4*)(gamma_f + idx[i] * 8), g1 = *(const float4*)(gamma_f + idx[i] * 8 + 4);
        const float4 b0 = *(const float4*)(beta_f + idx[i] * 8), b1 = *(const float4*)(beta_f + idx[i] * 8 + 4);
        const float g[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
        const float b[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            f[i][e] = __builtin_fmaf((f[i][e] - mean) * rstd, g[e], b[e]);
            m = __builtin_fmaxf(m, __builtin_fabsf(f[i][e]));
        }
    }
    m = wave_max(m);
    if ((threadIdx.x & 63) == 0) wmax[wave] = m;
    __syncthreads();
    float a = w8 < waves ? wmax[w8] : 0.0f;
    a = __builtin_fmaxf(a, lane_xor<4>(a));
    a = __builtin_fmaxf(a, lane_xor<2>(a));
    a = __builtin_fmaxf(a, lane_xor<1>(a));
    const float r = a > 0.0f ? 127.0f / a : 0.0f;
    if (threadIdx.x == 0) scale[row] = a / 127.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        uint32_t codes[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) codes[e] = code_bits(f[i][e] * r);
        if ((int)threadIdx.x + i * nt < nvec) __builtin_nontemporal_store(pack8(codes), (v2u*)code_dst(xq, row, idx[i] * 8, c_i, tiled));
    }
}

// One row per wave (hidden sizes up to 2048, where it measures faster than a workgroup per row): the three
// reductions are cross-lane shuffles, no barriers, and a lane keeps NV 16-byte loads in flight.
template <bool BF16, int NV>
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
                f[i][e] = (f[i][e] - mean) * rstd * g[e] + b[e];
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
    // Measured choice: up to 2048 channels one row per wave; wider rows a workgroup of as many threads as the row has vectors
    // for at NV per thread.  Few rows: short threads, the row's latency counts (1 x 5120 with 2 / 4 vectors 3.2 / 3.9 us,
    // 1024 x 9216 with 3 / 4 / 5 8.7 / 9.5 / 9.6).  Many rows: the reductions are shared by more elements of a wave
    // (4096 x 9216 with 3 / 5 / 6 vectors 34.1 / 34.8 / 31.5 us, 4096 x 5120 with 2 / 5 / 6 20.8 / 18.8 / 20.1, 8192 x 4096 with
    // 3 / 4 / 5 31.7 / 28.3 / 28.6).  With three exchanges, loads under a condition and 3 x 512 threads: 37.8 us at 4096 x 9216,
    // 11.9 at 1024 x 9216, 4.1 at 1 x 5120.
#define SQ_LN(BF, NV) sq_launch((ln_quant_kernel<BF, NV>), dim3((unsigned)t), dim3((unsigned)(((nvec + NV - 1) / NV + 63) / 64 * 64)), 0, st, xp, (int)c_i, gamma_f, beta_f, eps, scale, xq, tiled)
#define SQ_LNW(BF, NV) sq_launch((ln_quant_wave_kernel<BF, NV>), dim3((unsigned)((t + 3) / 4)), dim3(256), 0, st, xp, t, (int)c_i, gamma_f, beta_f, eps, scale, xq, tiled)
    const int nv = t >= 2048 ? (nvec <= 512 ? 4 : nvec <= 768 ? 5 : 6) : (nvec <= 640 ? 2 : nvec <= 1536 ? 3 : 4);
#define SQ_LNB(BF) do { switch (nv) { case 2: SQ_LN(BF, 2); break; case 3: SQ_LN(BF, 3); break; case 4: SQ_LN(BF, 4); break; case 5: SQ_LN(BF, 5); break; default: SQ_LN(BF, 6); break; } } while (0)
    if (dtype == SQ_BF16) {
        if (nvec <= 128) SQ_LNW(true, 2); else if (nvec <= 256) SQ_LNW(true, 4); else SQ_LNB(true);
    } else {
        if (nvec <= 128) SQ_LNW(false, 2); else if (nvec <= 256) SQ_LNW(false, 4); else SQ_LNB(false);
    }
#undef SQ_LN
#undef SQ_LNW
    return sq_launch_status();
}

}  // extern "C"
