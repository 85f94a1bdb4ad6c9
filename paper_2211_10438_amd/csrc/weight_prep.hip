// Offline weight preparation, gfx950: the statistics of Eq. 4, the smoothed weight of Eq. 3 and its
// per-tensor quantization by Eq. 1, written transposed ([C_o, C_i], contraction index contiguous)
// for the GEMM.  HBM bound: W is read once per statistic and once for its codes.
#include "common.h"

namespace {

template <bool BF16> SQ_DEVICE void unpack8w(const v4u raw, float (&f)[8])
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        f[2 * e] = load16_bits<BF16>(raw[e]);
        f[2 * e + 1] = load16_bits<BF16>(raw[e] >> 16);
    }
}

constexpr int kTensorParts = 512;  // most workgroups that leave a part of the tensor's maximum

// Maxima over rows of W: one row (input channel j) per WPR waves, four 16-byte loads per lane in flight.  ROWS: row_out[j] =
// max_n |W_jn|.  Otherwise the maximum over the tensor, each row scaled by s_j: a workgroup keeps it over all its rows and leaves it in
// tensor_max[blockIdx.x], or (ATOMIC: a workspace too small for that) adds it to the cleared tensor_max[0] with one atomic: the integer
// order of the bit patterns of non-negative floats is the float order.  (Atomics on one cell take some 12 ns each, one
// after the other, and want it cleared: preparation per tensor of 768 x 3072 11.5 us, now 9.1; with the reduction below 4096 x 4096 25.5, now 20.7.)
template <bool BF16, bool ROWS, int WPR, bool ATOMIC>
__global__ __launch_bounds__(256) void weight_row_absmax_kernel(const uint16_t* __restrict__ w, int c_i, int c_o,
                                                               const float* __restrict__ s, float* row_out,
                                                               uint32_t* tensor_max)
{
    constexpr int RPW = 4 / WPR, NT = WPR * 64;  // rows per workgroup, threads per row
    __shared__ float red[4];
    const int lane = threadIdx.x & 63, tid = threadIdx.x & (NT - 1);
    const int nvec = c_o >> 3;
    float all = 0.0f;
    for (int64_t j = (int64_t)blockIdx.x * RPW + threadIdx.x / NT; j < c_i; j += (int64_t)gridDim.x * RPW) {
        const v4u* wr = (const v4u*)(w + j * c_o);
        const float sj = s ? s[j] : 1.0f;
        float m = 0.0f;
        for (int i0 = tid; i0 < nvec; i0 += 4 * NT) {
            v4u raw[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) raw[i] = wr[i0 + i * NT < nvec ? i0 + i * NT : i0];  // past the end: the first one again
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float f[8];
                unpack8w<BF16>(raw[i], f);
#pragma unroll
                for (int e = 0; e < 8; ++e) m = __builtin_fmaxf(m, __builtin_fabsf(s ? f[e] * sj : f[e]));
            }
        }
        if constexpr (ROWS) {
            m = wave_max(m);
            if constexpr (WPR == 4) {
                __syncthreads();  // (the loop's trips are the same for the whole workgroup)
                if (lane == 0) red[threadIdx.x >> 6] = m;
                __syncthreads();
                m = __builtin_fmaxf(__builtin_fmaxf(red[0], red[1]), __builtin_fmaxf(red[2], red[3]));
            }
            if (tid == 0) row_out[j] = m;
        } else {
            all = __builtin_fmaxf(all, m);
        }
    }
    if constexpr (!ROWS) {
        all = wave_max(all);
        if (lane == 0) red[threadIdx.x >> 6] = all;
        __syncthreads();
        if (threadIdx.x == 0) {
            const uint32_t bits = __builtin_bit_cast(uint32_t, __builtin_fmaxf(__builtin_fmaxf(red[0], red[1]), __builtin_fmaxf(red[2], red[3])));
            if constexpr (ATOMIC) atomicMax(tensor_max, bits);
            else tensor_max[blockIdx.x] = bits;
        }
    }
}

__global__ void zero_u32_kernel(uint32_t* p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = 0u;
}

typedef float f4w __attribute__((ext_vector_type(4), aligned(4)));  // (a workspace need not be aligned to more than its words)

// Per-output-channel maxima of a slab of rows: out[slab][n] = max_j |W_jn * s_j|.  A workgroup owns 512 columns (a wave's row of 1 KB)
// over a slab, one row in four per wave with eight loads in flight; the waves meet in LDS.  The slabs' maxima go to memory by plain
// stores and meet in the kernel below.  (One atomic per slab and column leaves the XCD's L2 for the memory side: preparation per channel of
// 4096 x 4096 34.9 us, now 25; 5120 x 20480 99,
// now 92; 12288 x 64 39, now 13.7.  Eight loads in flight instead of four are 3 to 5 % of the large ones.)
template <bool BF16>
__global__ __launch_bounds__(256) void weight_col_absmax_kernel(const uint16_t* __restrict__ w, int c_i, int c_o,
                                                               const float* __restrict__ s, int rows_per_wg, float* out)
{
    __shared__ float red[3][512];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = (blockIdx.x * 64 + lane) * 8;
    const int j0 = blockIdx.y * rows_per_wg, j1 = c_i - j0 < rows_per_wg ? c_i : j0 + rows_per_wg;
    float m[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (n < c_o) {  // c_o % 8 == 0
        for (int j = j0 + wave; j < j1; j += 32) {
            v4u raw[8];
            float sj[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int jj = j + i * 4 < j1 ? j + i * 4 : j;  // past the end: the first row again
                raw[i] = *(const v4u*)(w + (int64_t)jj * c_o + n);
                sj[i] = s ? s[jj] : 1.0f;
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                float f[8];
                unpack8w<BF16>(raw[i], f);
#pragma unroll
                for (int e = 0; e < 8; ++e) m[e] = __builtin_fmaxf(m[e], __builtin_fabsf(s ? f[e] * sj[i] : f[e]));
            }
        }
    }
    if (wave > 0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) red[wave - 1][e * 64 + lane] = m[e];
    }
    __syncthreads();
    if (wave == 0 && n < c_o) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            m[e] = __builtin_fmaxf(__builtin_fmaxf(m[e], red[0][e * 64 + lane]), __builtin_fmaxf(red[1][e * 64 + lane], red[2][e * 64 + lane]));
        float* dst = out + (int64_t)blockIdx.y * c_o + n;
        *(f4w*)dst = f4w{m[0], m[1], m[2], m[3]};
        *(f4w*)(dst + 4) = f4w{m[4], m[5], m[6], m[7]};
    }
}

// The parts of the tensor's maximum to their largest, in place: behind more than 256 of them.  (Every wave of the transposing kernel reads
// the parts in front of its work.  Up to 256 that costs less than this launch -- 1024 x 8192 14.7 us without, 15.6 with it, 1536 x 1536
// 9.9 / 9.7 --, at 512 a tenth of that kernel: 6432 x 8104 70.3 / 68.4, 10368 x 13984 161.6 / 156.7, 5120 x 20480 tiled 90.6 / 88.6.)
__global__ __launch_bounds__(kTensorParts) void weight_parts_reduce_kernel(uint32_t* tensor_max, int parts)
{
    __shared__ float red[kTensorParts / 64];
    float a = wave_max(__builtin_bit_cast(float, tensor_max[(int)threadIdx.x < parts ? threadIdx.x : 0]));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = a;
    __syncthreads();  // everyone has read
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 1; i < kTensorParts / 64; ++i) a = __builtin_fmaxf(a, red[i]);
        tensor_max[0] = __builtin_bit_cast(uint32_t, a);
    }
}

// col_max[n] = the largest of part[slab][n].  Sixteen threads take the slabs of four columns, so that a slab is one load away for up to
// sixteen of them (one thread for all slabs of its columns: preparation of 12288 x 64 20.7 us, now 13.7; 944 x 40 14.6, now 13.4; 832 x 1032
// 15.8, now 15.1; 4096 x 4096 30.0, now 25.8).
__global__ __launch_bounds__(256) void weight_col_reduce_kernel(const float* part, int c_o, int slabs, float* col_max)
{
    __shared__ float4 red[16][16];
    const int quad = threadIdx.x & 15, first = threadIdx.x >> 4;
    const int n = (blockIdx.x * 16 + quad) * 4;
    float4 m = {0.0f, 0.0f, 0.0f, 0.0f};
    auto larger = [](float4 a, float4 b) { return float4{__builtin_fmaxf(a.x, b.x), __builtin_fmaxf(a.y, b.y), __builtin_fmaxf(a.z, b.z), __builtin_fmaxf(a.w, b.w)}; };
    if (n < c_o) {  // c_o % 8 == 0
#pragma unroll 4
        for (int s = first; s < slabs; s += 16) m = larger(m, *(const float4*)(part + (int64_t)s * c_o + n));
    }
    red[first][quad] = m;
    __syncthreads();
    if (first == 0 && n < c_o) {
#pragma unroll
        for (int i = 1; i < 16; ++i) m = larger(m, red[i][quad]);
        *(f4w*)(col_max + n) = f4w{m.x, m.y, m.z, m.w};
    }
}

// Quantize and transpose.  A wave owns 64 input x 128 output channels: lane (ng, jc) loads rows 16 jc .. 16 jc + 15 of its 8
// columns with sixteen 16-byte loads (256 contiguous bytes of a row per 16 lanes), quantizes them and packs four
// rows' codes into a word with byte permutes, so that it ends up with one 16-byte chunk (16 input channels of one output
// channel) per column.  The chunks pass through an LDS image of the wave's own, laid out like the tiled blocks (no workgroup
// barrier), and leave as whole 1 KB blocks (or 64-byte row segments).  The step of a column is formed once per 16 codes.
// (A byte-wise transpose of 64 x 64 tiles, a division per code with per-channel steps, took 83 us at 5120 x 20480.)
template <bool BF16>
__global__ __launch_bounds__(256) void weight_quant_transpose_kernel(const uint16_t* __restrict__ w, int c_i, int c_o,
                                                                    const float* __restrict__ s,
                                                                    const uint32_t* amax_bits, int parts, float* w_scale,
                                                                    int8_t* __restrict__ wq, bool tiled, bool per_channel)
{
    __shared__ __attribute__((aligned(1024))) char image[4][8192];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ng = lane & 15, jc = lane >> 4;
    const int n0 = blockIdx.x * 128, j0 = (blockIdx.y * 4 + wave) * 64;
    if (j0 >= c_i) return;
    const int n = n0 + ng * 8, j = j0 + jc * 16;
    const bool valid = n < c_o && j < c_i;  // c_o % 8 == 0, c_i % 16 == 0: a lane's piece is inside or outside as a whole
    float r[8];
    if (per_channel) {  // amax_bits[n]: maximum of column n
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float a = n < c_o ? __builtin_bit_cast(float, amax_bits[n + e]) : 0.0f;
            r[e] = a > 0.0f ? 127.0f / a : 0.0f;
            if (j0 == 0 && jc == 0 && n < c_o) w_scale[n + e] = a / 127.0f;
        }
    } else {
        float a;
        if (parts == 1) {
            a = __builtin_bit_cast(float, amax_bits[0]);
        } else {
            a = 0.0f;  // the largest of the parts
            for (int i = lane; i < parts; i += 64) a = __builtin_fmaxf(a, __builtin_bit_cast(float, amax_bits[i]));
            a = wave_max(a);
        }
        const float r0 = a > 0.0f ? 127.0f / a : 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) r[e] = r0;
        if (n0 == 0 && j0 == 0 && lane == 0) w_scale[0] = a / 127.0f;
    }
    v4u raw[16];
    float sj[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        raw[i] = valid ? __builtin_nontemporal_load((const v4u*)(w + (int64_t)(j + i) * c_o + n)) : v4u{0, 0, 0, 0};
        sj[i] = s && valid ? s[j + i] : 1.0f;
    }
    v4u out[8];  // the 16 codes of column e
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float f[4][8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            unpack8w<BF16>(raw[4 * q + i], f[i]);
            if (s) {
#pragma unroll
                for (int e = 0; e < 8; ++e) f[i][e] = f[i][e] * sj[4 * q + i];
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e)
            out[e][q] = pack4_low_bytes(code_bits(f[0][e] * r[e]), code_bits(f[1][e] * r[e]), code_bits(f[2][e] * r[e]), code_bits(f[3][e] * r[e]));
    }
    // image: block ng / 2 of 16 output channels, row 8 (ng & 1) + e, chunk jc at position jc ^ sw(row)
    auto sw = [](int row) { return ((row >> 1) & 3) ^ ((row >> 3) & 1); };
    char* img = image[wave];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int row = (ng & 1) * 8 + e;
        *(v4u*)(img + (ng >> 1) * 1024 + row * 64 + ((jc ^ sw(row)) << 4)) = out[e];
    }
    __builtin_amdgcn_wave_barrier();  // LDS serves one wave's accesses in order; keep the compiler from reordering
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const v4u val = *(const v4u*)(img + b * 1024 + lane * 16);
        const int nb = n0 + b * 16;
        if (nb >= c_o) break;
        if (tiled) {  // (rows of the last block beyond c_o: padding)
            __builtin_nontemporal_store(val, (v4u*)(wq + ((int64_t)(nb >> 4) * (c_i >> 6) + (j0 >> 6)) * 1024 + lane * 16));
        } else {
            const int row = lane >> 2, jj = j0 + (((lane & 3) ^ sw(row)) << 4);
            if (nb + row < c_o && jj < c_i) *(v4u*)(wq + (int64_t)(nb + row) * c_i + jj) = val;
        }
    }
}

// One wave per row, except where that leaves SIMDs without a wave and the rows are long enough for four (us, one wave / four
// waves per row): statistic of 64 x 20480 5.3 / 3.4, 256 x 12288 4.2 / 3.2, 768 x 20480 8.1 / 7.3, 1024 x 50272 23.1 / 18.1,
// but 768 x 4096 3.0 / 3.3, 1536 x 12288 7.7 / 8.0.  With the tensor's maximum every workgroup ends in an atomic on one cell, and
// the line lies lower (whole preparation): 256 x 20480 18.2 / 15.8, 64 x 50272 24.8 / 14.9, but 256 x 8192 12.3 / 13.4, 768 x
// 20480 24.4 / 28.9.
// `room`: cells of tensor_max.  Returns the parts the tensor's maximum is left in (1 where they met by atomics, or for ROWS).
template <bool ROWS>
int launch_row_absmax(const uint16_t* w, sq_dtype dtype, int c_i, int c_o, const float* s, float* row_out, uint32_t* tensor_max, size_t room, hipStream_t st)
{
    const bool wide = ROWS ? c_i <= 1024 && c_o > 4096 : c_i <= 256 && c_o > 16384;
    const int64_t need = wide ? c_i : ((int64_t)c_i + 3) / 4, cap = ROWS ? 65535 : kTensorParts;  // (the kernel strides over the rest)
    const dim3 grid((unsigned)(need < cap ? need : cap));
    const bool atomic = !ROWS && room < grid.x;
    if (atomic) sq_launch(zero_u32_kernel, dim3(1), dim3(256), 0, st, tensor_max, (int64_t)1);
#define SQ_ROW(BF, WPR)                                                                                                                    \
    do {                                                                                                                                   \
        if (atomic) sq_launch((weight_row_absmax_kernel<BF, ROWS, WPR, !ROWS>), grid, dim3(256), 0, st, w, c_i, c_o, s, row_out, tensor_max); \
        else sq_launch((weight_row_absmax_kernel<BF, ROWS, WPR, false>), grid, dim3(256), 0, st, w, c_i, c_o, s, row_out, tensor_max);       \
    } while (0)
    if (dtype == SQ_BF16) {
        if (wide) SQ_ROW(true, 4); else SQ_ROW(true, 1);
    } else {
        if (wide) SQ_ROW(false, 4); else SQ_ROW(false, 1);
    }
#undef SQ_ROW
    return ROWS || atomic ? 1 : (int)grid.x;
}

}  // namespace

extern "C" {

sq_status sq_weight_absmax_per_in_channel(const void* w, sq_dtype dtype, int64_t c_i, int64_t c_o, float* out,
                                          void* stream)
{
    if (!w || !out) return SQ_ERR_NULL;
    if (c_i <= 0 || c_o <= 0 || c_i >= ((int64_t)1 << 31) || c_o >= ((int64_t)1 << 31)) return SQ_ERR_SHAPE;
    if (dtype != SQ_F16 && dtype != SQ_BF16) return SQ_ERR_UNSUPPORTED;
    if ((c_o & 7) || !sq_aligned16(w)) return SQ_ERR_ALIGN;
    launch_row_absmax<true>((const uint16_t*)w, dtype, (int)c_i, (int)c_o, nullptr, out, nullptr, 0, (hipStream_t)stream);
    return sq_launch_status();
}

sq_status sq_prepare_weight(const void* w, sq_dtype dtype, const float* s, int64_t c_i, int64_t c_o, int8_t* wq,
                            sq_layout wq_layout, float* w_scale, int w_scale_per_channel, void* workspace, size_t ws_bytes,
                            void* stream)
{
    if (!w || !wq || !w_scale) return SQ_ERR_NULL;
    if (c_i <= 0 || c_o <= 0 || c_i >= ((int64_t)1 << 31) || c_o >= ((int64_t)1 << 31)) return SQ_ERR_SHAPE;
    if (dtype != SQ_F16 && dtype != SQ_BF16) return SQ_ERR_UNSUPPORTED;
    if (wq_layout != SQ_ROW_MAJOR && wq_layout != SQ_TILED) return SQ_ERR_UNSUPPORTED;
    if ((c_i & 15) || (c_o & 7) || !sq_aligned16(w) || !sq_aligned16(wq)) return SQ_ERR_ALIGN;
    if (wq_layout == SQ_TILED && (c_i & 63)) return SQ_ERR_ALIGN;
    const bool tiled = wq_layout == SQ_TILED;
    const bool pc = w_scale_per_channel != 0;
    if (!workspace || ws_bytes < sizeof(uint32_t) * (pc ? (size_t)c_o : 1)) return SQ_ERR_WORKSPACE;
    if (((int64_t)((c_i + 63) / 64)) > 65535) return SQ_ERR_SHAPE;
    hipStream_t st = (hipStream_t)stream;
    uint32_t* amax = (uint32_t*)workspace;
    const dim3 grid2((unsigned)((c_o + 127) / 128), (unsigned)((c_i + 255) / 256));
    int parts = 1;
    if (pc) {
        // about four workgroups per compute unit, slabs of at least 64 rows.  The slabs' maxima wait in the code buffer, which is
        // written last and has room: 4 bytes per column and slab of 64 rows or more against one per weight.
        const int64_t colb = (c_o / 8 + 63) / 64;
        int64_t slabs = (1024 + colb - 1) / colb;
        if (slabs > (c_i + 63) / 64) slabs = (c_i + 63) / 64;
        if (c_i <= 96) slabs = 1;  // no second launch (us, two slabs / one: 80 x 576 13.4 / 12.8, 128 x 576 13.2 / 14.2)
        const int rows = (int)((c_i + slabs - 1) / slabs);
        slabs = (c_i + rows - 1) / rows;
        float* part = slabs > 1 ? (float*)wq : (float*)amax;
        const dim3 gridc((unsigned)colb, (unsigned)slabs);
        if (dtype == SQ_BF16) sq_launch(weight_col_absmax_kernel<true>, gridc, dim3(256), 0, st, (const uint16_t*)w, (int)c_i, (int)c_o, s, rows, part);
        else sq_launch(weight_col_absmax_kernel<false>, gridc, dim3(256), 0, st, (const uint16_t*)w, (int)c_i, (int)c_o, s, rows, part);
        if (slabs > 1) sq_launch(weight_col_reduce_kernel, dim3((unsigned)((c_o / 4 + 15) / 16)), dim3(256), 0, st, part, (int)c_o, (int)slabs, (float*)amax);
    } else {
        parts = launch_row_absmax<false>((const uint16_t*)w, dtype, (int)c_i, (int)c_o, s, nullptr, amax, ws_bytes / sizeof(uint32_t), st);
        if (parts > 256) {
            sq_launch(weight_parts_reduce_kernel, dim3(1), dim3(kTensorParts), 0, st, amax, parts);
            parts = 1;
        }
    }
    if (dtype == SQ_BF16) sq_launch(weight_quant_transpose_kernel<true>, grid2, dim3(256), 0, st, (const uint16_t*)w, (int)c_i, (int)c_o, s, amax, parts, w_scale, wq, tiled, pc);
    else sq_launch(weight_quant_transpose_kernel<false>, grid2, dim3(256), 0, st, (const uint16_t*)w, (int)c_i, (int)c_o, s, amax, parts, w_scale, wq, tiled, pc);
    return sq_launch_status();
}

}  // extern "C"
