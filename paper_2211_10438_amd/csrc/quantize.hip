// Activation quantization (Eq. 1) at the granularities of Table 2, gfx950.
//
// Per-token dynamic (O1): one pass over HBM.  A row lives in registers between the absmax
// reduction and the rounding, so the traffic is 2 B read + 1 B written per element.  Rows are
// handled by a 256-thread workgroup (wide rows) or by one 64-lane wave (narrow rows, reduction
// with cross-lane shuffles only).
// Per-tensor static (O3): pure elementwise pass, saturating.
// Per-tensor dynamic (O2): tensors that one workgroup or a few can read whole take one launch; larger ones two (partial maxima,
// quantize; the second read is served by the memory-side cache), callers with a small workspace three (clear, absmax with
// atomic max on the float's bit pattern, quantize); results are identical.
#include <type_traits>

#include "common.h"

namespace {

template <bool BF16> SQ_DEVICE void unpack8(const v4u raw, float (&f)[8])
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        f[2 * e] = load16_bits<BF16>(raw[e]);
        f[2 * e + 1] = load16_bits<BF16>(raw[e] >> 16);
    }
}

// x_hat = fl32(x * inv_s_j) for the 8 channels starting at `col` (Eq. 3 applied to the activation).
SQ_DEVICE void smooth8(float (&f)[8], const float* inv_s, int col)
{
    const float4 a = *(const float4*)(inv_s + col);
    const float4 b = *(const float4*)(inv_s + col + 4);
    f[0] = f[0] * a.x; f[1] = f[1] * a.y; f[2] = f[2] * a.z; f[3] = f[3] * a.w;
    f[4] = f[4] * b.x; f[5] = f[5] * b.y; f[6] = f[6] * b.z; f[7] = f[7] * b.w;
}

SQ_DEVICE float absmax8(const float (&f)[8])
{
    float m = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) m = __builtin_fmaxf(m, __builtin_fabsf(f[e]));
    return m;
}

SQ_DEVICE v2u quant8(const float (&f)[8], float r)
{
    v2u out;
#pragma unroll
    for (int h = 0; h < 2; ++h)
        out[h] = pack4_low_bytes(code_bits(f[4 * h] * r), code_bits(f[4 * h + 1] * r), code_bits(f[4 * h + 2] * r),
                                 code_bits(f[4 * h + 3] * r));
    return out;
}

// Block-wide max for a workgroup of NT threads (NT / 64 waves).
template <int NT> SQ_DEVICE float block_max(float v, float* red)
{
    v = wave_max(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    float m = red[0];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) m = __builtin_fmaxf(m, red[w]);
    return m;
}
SQ_DEVICE float block_max_256(float v, float* red) { return block_max<256>(v, red); }

// One row per workgroup of NT threads; NV 16-byte vectors (8 elements) per thread kept in registers.
// KEEP: the smoothed fp32 values stay in registers between the two phases (worth it while NV is small);
// otherwise x * inv_s is evaluated again in the second phase -- the same fp32 product, hence the same code.
template <bool BF16, int NV, int NT, bool KEEP>
__global__ __launch_bounds__(NT) void quant_per_token_block(const uint16_t* __restrict__ x, int64_t ldx, int c_i,
                                                           const float* __restrict__ inv_s, float* __restrict__ scale,
                                                           int8_t* __restrict__ xq, bool tiled)
{
    __shared__ float red[NT / 64];
    const int64_t row = blockIdx.x;
    const v4u* xr = (const v4u*)(x + row * ldx);
    const int nvec = c_i >> 3;
    v4u raw[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = threadIdx.x + i * NT;
        raw[i] = idx < nvec ? __builtin_nontemporal_load(xr + idx) : v4u{0, 0, 0, 0};
    }
    float kept[KEEP ? NV : 1][8];
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = threadIdx.x + i * NT;
        float f[8];
        unpack8<BF16>(raw[i], f);
        if (inv_s && idx < nvec) smooth8(f, inv_s, idx * 8);
        m = __builtin_fmaxf(m, absmax8(f));
        if constexpr (KEEP) {
#pragma unroll
            for (int e = 0; e < 8; ++e) kept[i][e] = f[e];
        }
    }
    const float a = block_max<NT>(m, red);
    const float r = a > 0.0f ? 127.0f / a : 0.0f;
    if (threadIdx.x == 0) scale[row] = a / 127.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = threadIdx.x + i * NT;
        if (idx < nvec) {
            float f[8];
            if constexpr (KEEP) {
#pragma unroll
                for (int e = 0; e < 8; ++e) f[e] = kept[i][e];
            } else {
                unpack8<BF16>(raw[i], f);
                if (inv_s) smooth8(f, inv_s, idx * 8);
            }
            __builtin_nontemporal_store(quant8(f, r), (v2u*)code_dst(xq, row, idx * 8, c_i, tiled));
        }
    }
}

// Two rows per workgroup for inputs that take smoothing factors: the 4 * c_i bytes of fp32 factors a row needs are
// twice the row's own 2 * c_i bytes, so reading them once for two rows takes a third off what a workgroup pulls
// through its compute unit.  Both rows are in flight together (not one after the other), the products x * inv_s stay
// in registers between the reduction and the rounding.
template <bool BF16, int NV, int NT>
__global__ __launch_bounds__(NT) void quant_per_token_block2(const uint16_t* __restrict__ x, int64_t ldx, int c_i, int64_t t,
                                                            const float* __restrict__ inv_s, float* __restrict__ scale,
                                                            int8_t* __restrict__ xq, bool tiled)
{
    __shared__ float red[2][NT / 64];
    const int64_t row0 = (int64_t)blockIdx.x * 2;
    const bool two = row0 + 1 < t;
    const v4u* xr0 = (const v4u*)(x + row0 * ldx);
    const v4u* xr1 = (const v4u*)(x + (two ? row0 + 1 : row0) * ldx);
    const int nvec = c_i >> 3;
    v4u raw0[NV], raw1[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = threadIdx.x + i * NT;
        raw0[i] = idx < nvec ? __builtin_nontemporal_load(xr0 + idx) : v4u{0, 0, 0, 0};
        raw1[i] = idx < nvec ? __builtin_nontemporal_load(xr1 + idx) : v4u{0, 0, 0, 0};
    }
    float k0[NV][8], k1[NV][8];
    float m0 = 0.0f, m1 = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = threadIdx.x + i * NT;
        unpack8<BF16>(raw0[i], k0[i]);
        unpack8<BF16>(raw1[i], k1[i]);
        if (idx < nvec) {
            const float4 a = *(const float4*)(inv_s + idx * 8);
            const float4 b = *(const float4*)(inv_s + idx * 8 + 4);
            const float s8[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                k0[i][e] = k0[i][e] * s8[e];
                k1[i][e] = k1[i][e] * s8[e];
            }
        }
        m0 = __builtin_fmaxf(m0, absmax8(k0[i]));
        m1 = __builtin_fmaxf(m1, absmax8(k1[i]));
    }
    m0 = wave_max(m0);
    m1 = wave_max(m1);
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = m0;
        red[1][threadIdx.x >> 6] = m1;
    }
    __syncthreads();
    float a0 = red[0][0], a1 = red[1][0];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) {
        a0 = __builtin_fmaxf(a0, red[0][w]);
        a1 = __builtin_fmaxf(a1, red[1][w]);
    }
    const float r0 = a0 > 0.0f ? 127.0f / a0 : 0.0f, r1 = a1 > 0.0f ? 127.0f / a1 : 0.0f;
    if (threadIdx.x == 0) {
        scale[row0] = a0 / 127.0f;
        if (two) scale[row0 + 1] = a1 / 127.0f;
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = threadIdx.x + i * NT;
        if (idx < nvec) {
            __builtin_nontemporal_store(quant8(k0[i], r0), (v2u*)code_dst(xq, row0, idx * 8, c_i, tiled));
            if (two) __builtin_nontemporal_store(quant8(k1[i], r1), (v2u*)code_dst(xq, row0 + 1, idx * 8, c_i, tiled));
        }
    }
}

// One row per wave (4 rows per workgroup): for narrow rows.
template <bool BF16, int NV>
__global__ __launch_bounds__(256) void quant_per_token_wave(const uint16_t* __restrict__ x, int64_t ldx, int c_i, int64_t t,
                                                           const float* __restrict__ inv_s, float* __restrict__ scale,
                                                           int8_t* __restrict__ xq, bool tiled)
{
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= t) return;
    const v4u* xr = (const v4u*)(x + row * ldx);
    const int nvec = c_i >> 3;
    v4u raw[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = lane + i * 64;
        raw[i] = idx < nvec ? xr[idx] : v4u{0, 0, 0, 0};
    }
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = lane + i * 64;
        float f[8];
        unpack8<BF16>(raw[i], f);
        if (inv_s && idx < nvec) smooth8(f, inv_s, idx * 8);
        m = __builtin_fmaxf(m, absmax8(f));
    }
    const float a = wave_max(m);
    const float r = a > 0.0f ? 127.0f / a : 0.0f;
    if (lane == 0) scale[row] = a / 127.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = lane + i * 64;
        if (idx < nvec) {
            float f[8];
            unpack8<BF16>(raw[i], f);
            if (inv_s) smooth8(f, inv_s, idx * 8);
            *(v2u*)code_dst(xq, row, idx * 8, c_i, tiled) = quant8(f, r);
        }
    }
}

// Rows wider than the register-resident variants cover: two passes over the row (second one is
// served by the caches for any realistic width).
template <bool BF16>
__global__ __launch_bounds__(256) void quant_per_token_stream(const uint16_t* __restrict__ x, int64_t ldx, int c_i,
                                                             const float* __restrict__ inv_s, float* __restrict__ scale,
                                                             int8_t* __restrict__ xq, bool tiled)
{
    __shared__ float red[4];
    const int64_t row = blockIdx.x;
    const v4u* xr = (const v4u*)(x + row * ldx);
    const int nvec = c_i >> 3;
    float m = 0.0f;
    for (int idx = threadIdx.x; idx < nvec; idx += 256) {
        float f[8];
        unpack8<BF16>(xr[idx], f);
        if (inv_s) smooth8(f, inv_s, idx * 8);
        m = __builtin_fmaxf(m, absmax8(f));
    }
    const float a = block_max_256(m, red);
    const float r = a > 0.0f ? 127.0f / a : 0.0f;
    if (threadIdx.x == 0) scale[row] = a / 127.0f;
    for (int idx = threadIdx.x; idx < nvec; idx += 256) {
        float f[8];
        unpack8<BF16>(xr[idx], f);
        if (inv_s) smooth8(f, inv_s, idx * 8);
        *(v2u*)code_dst(xq, row, idx * 8, c_i, tiled) = quant8(f, r);
    }
}

// ---- per-tensor

__global__ void fill_u32_kernel(uint32_t* p, uint32_t v, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// The per-tensor kernels number the 16-byte vectors of the whole [t, c_i] tensor and find row and column of each by a
// division.  Below 2^31 vectors (34 GB of activations) it is a multiply-high and a shift (exact: d >= 2, n < 2^31, m the
// reciprocal rounded up); the 64-bit division it replaces is some 40 instructions per vector, which is what an 8-element
// vector's whole quantization costs.  Larger tensors (WIDE) keep the 64-bit form.
struct RowOf {
    uint32_t nvec, mul, shift;
    template <bool WIDE> __device__ __forceinline__ int64_t row(int64_t g) const
    {
        if constexpr (WIDE) return g / (int64_t)nvec;
        else return (int64_t)(__umulhi((uint32_t)g, mul) >> shift);
    }
};
RowOf row_of(int64_t nvec)
{
    uint32_t l = 1;
    while (((int64_t)1 << l) < nvec) ++l;  // 2^(l-1) < nvec <= 2^l (c_i % 16 == 0: nvec >= 2)
    return RowOf{(uint32_t)nvec, (uint32_t)((((uint64_t)1 << (31 + l)) / (uint64_t)nvec) + 1), l - 1};
}

// absmax over the whole [t, c_i] tensor.  Every workgroup takes one contiguous range of vectors, four 16-byte loads per
// thread in flight, and leaves its maximum in partial[blockIdx.x]: a plain store, nothing to clear beforehand.  (Same-
// address atomics serialize at about 12 ns: one per workgroup of a 4096-workgroup grid made this pass 49 us on a
// 1000 x 9216 tensor whose 18 MB take 4; the whole quantization of that tensor went from 57 to 15 us, of 2048 x 12288 from
// 66 to 25, of 2048 x 49152 from 110 to 83.)  With ATOMIC (scratch of a few bytes only) the maxima meet in partial[0], which
// the caller has cleared: the integer order of the bit patterns of non-negative floats is the float order.
constexpr int kAbsmaxThreads = 512, kAbsmaxUnroll = 4;
template <bool BF16, bool WIDE, bool ATOMIC>
__global__ __launch_bounds__(kAbsmaxThreads) void tensor_absmax_kernel(const uint16_t* __restrict__ x, int64_t ldx, RowOf ro, int64_t total,
                                                                      int64_t per_wg, const float* __restrict__ inv_s, uint32_t* partial)
{
    constexpr int NT = kAbsmaxThreads, U = kAbsmaxUnroll;
    __shared__ float red[NT / 64];
    const int64_t g0 = (int64_t)blockIdx.x * per_wg, g1 = g0 + per_wg < total ? g0 + per_wg : total;
    float m = 0.0f;
    // (whole rounds without bounds checks; in the last one a load that is not there costs less as a branch than as another copy of the last vector:
    // smoothed 4096 x 20480 both launches 81.4 / 80.0 us, 512 x 5120 7.1 / 6.9)
    auto vectors = [&](int64_t base, auto FULL_) {
        constexpr bool FULL = decltype(FULL_)::value;
        v4u raw[U];
        int col[U];
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int64_t g = base + i * NT;
            raw[i] = v4u{0, 0, 0, 0};
            col[i] = 0;
            if (FULL || g < g1) {
                const int64_t row = ro.row<WIDE>(g);
                const int idx = (int)(g - row * ro.nvec);
                raw[i] = ((const v4u*)(x + row * ldx))[idx];
                col[i] = idx * 8;
            }
        }
#pragma unroll
        for (int i = 0; i < U; ++i) {
            float f[8];
            unpack8<BF16>(raw[i], f);
            if (inv_s) smooth8(f, inv_s, col[i]);
            m = __builtin_fmaxf(m, absmax8(f));
        }
    };
    int64_t first = g0;
    for (; first + NT * U <= g1; first += NT * U) vectors(first + threadIdx.x, std::true_type{});
    if (first < g1) vectors(first + threadIdx.x, std::false_type{});
    m = block_max<NT>(m, red);
    if (threadIdx.x == 0) {
        if constexpr (ATOMIC) atomicMax(partial, __builtin_bit_cast(uint32_t, m));
        else partial[blockIdx.x] = __builtin_bit_cast(uint32_t, m);
    }
}

// Elementwise quantization with one step for the whole tensor, U vectors per thread in flight.  DYNAMIC: the step comes
// from the n_partial maxima of the absmax pass (and is written to scale[0]); otherwise scale[0] holds the calibrated Delta.
template <bool BF16, bool DYNAMIC, bool WIDE, int U>
__global__ __launch_bounds__(256) void quant_per_tensor_kernel(const uint16_t* __restrict__ x, int64_t ldx, int c_i, RowOf ro, int64_t total,
                                                              const float* __restrict__ inv_s, float* scale,
                                                              const uint32_t* partial, int n_partial, int8_t* __restrict__ xq, bool tiled)
{
    __shared__ float red[4];
    float r = 0.0f;
    bool have_r = false;
    for (int64_t base = (int64_t)blockIdx.x * (256 * U) + threadIdx.x; base - threadIdx.x < total; base += (int64_t)gridDim.x * (256 * U)) {
        v4u raw[U];
        int64_t row[U];
        int idx[U];
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int64_t g = base + i * 256;
            raw[i] = v4u{0, 0, 0, 0};
            row[i] = 0;
            idx[i] = 0;
            if (g < total) {
                row[i] = ro.row<WIDE>(g);
                idx[i] = (int)(g - row[i] * ro.nvec);
                raw[i] = __builtin_nontemporal_load((const v4u*)(x + row[i] * ldx) + idx[i]);
            }
        }
        if (!have_r) {  // behind the first loads, so that the two latencies overlap
            have_r = true;
            if constexpr (DYNAMIC) {
                float a = 0.0f;
                for (int i = threadIdx.x; i < n_partial; i += 256) a = __builtin_fmaxf(a, __builtin_bit_cast(float, partial[i]));
                a = block_max_256(a, red);
                r = a > 0.0f ? 127.0f / a : 0.0f;
                if (blockIdx.x == 0 && threadIdx.x == 0) scale[0] = a / 127.0f;
            } else {
                const float delta = scale[0];
                r = delta > 0.0f ? 1.0f / delta : 0.0f;
            }
        }
#pragma unroll
        for (int i = 0; i < U; ++i) {
            if (base + i * 256 < total) {
                float f[8];
                unpack8<BF16>(raw[i], f);
                if (inv_s) smooth8(f, inv_s, idx[i] * 8);
                __builtin_nontemporal_store(quant8(f, r), (v2u*)code_dst(xq, row[i], idx[i] * 8, c_i, tiled));
            }
        }
    }
}

constexpr int kO2Parts = 512;  // most partial maxima of a tensor

// A tensor that one workgroup holds in its registers: one launch.  A launch and a load's way from memory and back are the time (16 x 768
// 2.6 us, as two launches 4.6).  A grid that meets at an arrival count between maximum and rounding is not worth its wait at any size: 3 us
// and more for atomics, polls and the maxima's way through memory on top of one pass, where a second launch costs 2.5 (16 x 768 6.7 us,
// now 2.6; 64 x 4096 10.5, now 5.2; 333 x 5120 16.5, now 6.5).
template <bool BF16, int NV>
__global__ __launch_bounds__(1024) void quant_per_tensor_small_kernel(const uint16_t* __restrict__ x, int64_t ldx, int c_i, RowOf ro, int total,
                                                                     const float* __restrict__ inv_s, float* scale, int8_t* __restrict__ xq, bool tiled)
{
    __shared__ float red[16];
    v4u raw[NV];
    int row[NV], col[NV];
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int g = (int)threadIdx.x + i * 1024 < total ? (int)threadIdx.x + i * 1024 : total - 1;  // past the end: the last one again
        row[i] = (int)ro.row<false>(g);
        const int idx = g - row[i] * (int)ro.nvec;
        raw[i] = __builtin_nontemporal_load((const v4u*)(x + row[i] * ldx) + idx);
        col[i] = idx * 8;
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        float f[8];
        unpack8<BF16>(raw[i], f);
        if (inv_s) smooth8(f, inv_s, col[i]);
        m = __builtin_fmaxf(m, absmax8(f));
    }
    const float a = block_max<1024>(m, red);
    const float r = a > 0.0f ? 127.0f / a : 0.0f;
    if (threadIdx.x == 0) scale[0] = a / 127.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        if ((int)threadIdx.x + i * 1024 < total) {
            float f[8];
            unpack8<BF16>(raw[i], f);
            if (inv_s) smooth8(f, inv_s, col[i]);
            __builtin_nontemporal_store(quant8(f, r), (v2u*)code_dst(xq, row[i], col[i], c_i, tiled));
        }
    }
}

// Somewhat larger tensors in one launch too: each of a few workgroups reads the whole tensor for its maximum (one pass through an L2 at some 40
// GB/s per compute unit) and quantizes one vector per thread.  us, this / the one workgroup above with four vectors per thread / two
// launches: 8 x 4096 3.1 / 3.6 / 4.3 (smoothed 3.7 / 4.6 / 4.9), 9 x 4096 3.4 / - / 4.3, 16 x 4096 4.0 / - / 4.3, 32 x 4096 6.2 / - / 4.4; smoothed, where
// every workgroup reads the factors too, 12 x 4096 5.2 / - / 4.8.  And a launch less of the host's time: calls one after the other 16 x 4096
// 5.9 / - / 8.7.
template <bool BF16>
__global__ __launch_bounds__(1024) void quant_per_tensor_shared_kernel(const uint16_t* __restrict__ x, int64_t ldx, int c_i, RowOf ro, int total,
                                                                      const float* __restrict__ inv_s, float* scale, int8_t* __restrict__ xq, bool tiled)
{
    constexpr int U = 4;  // loads in flight per thread
    __shared__ float red[16];
    auto load = [&](int g, v4u& raw, int& row, int& col) {
        const int at = g < total ? g : total - 1;  // past the end: the last one again
        row = (int)ro.row<false>(at);
        const int idx = at - row * (int)ro.nvec;
        raw = *((const v4u*)(x + row * ldx) + idx);
        col = idx * 8;
    };
    const int mine = (int)blockIdx.x * 1024 + (int)threadIdx.x;
    v4u own;
    int row, col;
    load(mine, own, row, col);
    float m = 0.0f;
    for (int base = threadIdx.x; base < total; base += 1024 * U) {
        v4u raw[U];
        int c[U], any_row;
#pragma unroll
        for (int i = 0; i < U; ++i) load(base + i * 1024, raw[i], any_row, c[i]);
#pragma unroll
        for (int i = 0; i < U; ++i) {
            float f[8];
            unpack8<BF16>(raw[i], f);
            if (inv_s) smooth8(f, inv_s, c[i]);
            m = __builtin_fmaxf(m, absmax8(f));
        }
    }
    const float a = block_max<1024>(m, red);
    const float r = a > 0.0f ? 127.0f / a : 0.0f;
    if (mine == 0) scale[0] = a / 127.0f;
    if (mine < total) {
        float f[8];
        unpack8<BF16>(own, f);
        if (inv_s) smooth8(f, inv_s, col);
        __builtin_nontemporal_store(quant8(f, r), (v2u*)code_dst(xq, row, col, c_i, tiled));
    }
}

// Per-channel calibration statistic: out_j = max_t |x_tj|.  A workgroup owns 64 neighbouring channels (one 128-byte line
// of a row: 8 lanes) and, 32 rows at a time with four rows per lane in flight, a range of rows; the row groups meet in LDS.
// While the row range is the whole batch (gridDim.y == 1) the result is stored as it is; longer batches are cut into row
// ranges whose maxima meet by atomic max on the bit patterns (cleared beforehand).  One atomic per channel and workgroup
// of two rows each, as this pass did before, took 53 us on a 512 x 5120 batch (5 MB; now 4.4), 91 on 2048 x 12288 (14.8), 146
// on 40000 x 5120 (99).
constexpr int kChannelRows = 32;
template <bool BF16>
__global__ __launch_bounds__(256) void act_absmax_per_channel_kernel(const uint16_t* __restrict__ x, int c_i, int64_t t, int64_t rows_per_wg,
                                                                    uint32_t* out_bits, int first)
{
    __shared__ float red[4][64];
    const int nvec = c_i >> 3;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = first + (int)blockIdx.x;  // 64-channel column
    const int idx = col * 8 + (threadIdx.x & 7);
    const int64_t r0 = (int64_t)blockIdx.y * rows_per_wg, r1 = r0 + rows_per_wg < t ? r0 + rows_per_wg : t;
    float m[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (idx < nvec) {
        for (int64_t row = r0 + (threadIdx.x >> 3); row < r1; row += 4 * kChannelRows) {
            v4u raw[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {  // past the end: the first row of this lane again
                const int64_t rr = row + i * kChannelRows < r1 ? row + i * kChannelRows : row;
                raw[i] = ((const v4u*)(x + rr * (int64_t)c_i))[idx];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float f[8];
                unpack8<BF16>(raw[i], f);
#pragma unroll
                for (int e = 0; e < 8; ++e) m[e] = __builtin_fmaxf(m[e], __builtin_fabsf(f[e]));
            }
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int o = 32; o >= 8; o >>= 1) m[e] = __builtin_fmaxf(m[e], __shfl_xor(m[e], o, 64));
    if (lane < 8) {
#pragma unroll
        for (int e = 0; e < 8; ++e) red[wave][lane * 8 + e] = m[e];
    }
    __syncthreads();
    const int64_t c = (int64_t)col * 64 + threadIdx.x;
    if (threadIdx.x < 64 && c < c_i) {
        const float v = __builtin_fmaxf(__builtin_fmaxf(red[0][threadIdx.x], red[1][threadIdx.x]),
                                        __builtin_fmaxf(red[2][threadIdx.x], red[3][threadIdx.x]));
        if (gridDim.y == 1) out_bits[c] = __builtin_bit_cast(uint32_t, v);
        else atomicMax(out_bits + c, __builtin_bit_cast(uint32_t, v));
    }
}

template <bool BF16>
void launch_per_token(const uint16_t* x, int64_t ldx, int c_i, int64_t t, const float* inv_s, float* scale, int8_t* xq,
                      bool tiled, hipStream_t st)
{
    const int nvec = c_i >> 3;
#define SQ_WAVE(NV) sq_launch((quant_per_token_wave<BF16, NV>), dim3((unsigned)((t + 3) / 4)), dim3(256), 0, st, x, ldx, c_i, t, inv_s, scale, xq, tiled)
#define SQ_BLOCK(NV, NT)                                                                                                        \
    do {                                                                                                                        \
        if (inv_s && NV <= 6) sq_launch((quant_per_token_block<BF16, NV, NT, true>), dim3((unsigned)t), dim3(NT), 0, st, x, ldx, c_i, inv_s, scale, xq, tiled); \
        else sq_launch((quant_per_token_block<BF16, NV, NT, false>), dim3((unsigned)t), dim3(NT), 0, st, x, ldx, c_i, inv_s, scale, xq, tiled);                 \
    } while (0)
    // Few rows: one vector per thread, the row's latency counts (1 x 5120 with smoothing factors 2.8 -> 2.3 us, 256 x 5120
    // 3.3 -> 2.9; with 1000 rows and more the fewer, longer threads below are ahead).
    if (t <= 256 && nvec > 256 && nvec <= 1024) SQ_BLOCK(1, 1024);
    else if (nvec <= 64) SQ_WAVE(1);
    else if (nvec <= 128) SQ_WAVE(2);
    else if (nvec <= 256) SQ_BLOCK(1, 256);
    else if (nvec <= 512) SQ_BLOCK(2, 256);
    else if (nvec <= 1024) SQ_BLOCK(4, 256);
    // workgroup sizes that divide the row evenly (every thread the same number of vectors) measure 4-12 % faster
    // than the next power of two: the hidden sizes 9216 and 12288 and the 36864-wide FFN of the former
    // (with smoothing factors the 12288-wide row takes two rows per workgroup: 18.6 against 20.9 us at 2048 rows;
    //  the 9216-wide row measured no gain from it)
    else if (nvec == 1536 && inv_s) sq_launch((quant_per_token_block2<BF16, 2, 768>), dim3((unsigned)((t + 1) / 2)), dim3(768), 0, st, x, ldx, c_i, t, inv_s, scale, xq, tiled);
    else if (nvec == 1152) SQ_BLOCK(2, 576);
    else if (nvec == 1536) SQ_BLOCK(2, 768);
    else if (nvec == 4608) SQ_BLOCK(6, 768);
    else if (nvec <= 2048) SQ_BLOCK(2, 1024);  // measured: from 8192 channels on, 1024 threads per row beat 256
    else if (nvec <= 4096) SQ_BLOCK(4, 1024);
    else if (nvec <= 6144) SQ_BLOCK(6, 1024);
    else if (nvec <= 8192) SQ_BLOCK(8, 1024);
    else sq_launch((quant_per_token_stream<BF16>), dim3((unsigned)t), dim3(256), 0, st, x, ldx, c_i, inv_s, scale, xq, tiled);
#undef SQ_WAVE
#undef SQ_BLOCK
}

// Vectors per thread of the elementwise pass, static mode measured on rotating buffers (rows / tiled codes): two from 2^21
// vectors on (2048 x 12288: 14.6 / 16.1 us against 15.5 / 15.1 with one and 16.0 / 18.1 with four; 2048 x 49152: 49 / 53
// against 56 / 55 and 54 / 58), one below (1000 x 9216: 7.0 / 7.3 us against 7.0 / 8.1 and 8.2 / 9.2).  With a dynamic step every
// workgroup reduces the partial maxima first, and fewer of them pay from 2^19 vectors on (both passes, one / two / four: 512 x 5120
// 7.1 / 7.2 / -, 512 x 9216 9.0 / 8.6 / 9.5, 512 x 12288 10.3 / 9.6 / 10.3, 1000 x 9216 12.8 / 12.4 / 13.3; each wave reducing them for itself, without
// a barrier, takes longer at every size).
template <bool BF16, bool DYNAMIC>
void launch_per_tensor(const uint16_t* x, int64_t ldx, int c_i, int64_t total, const float* inv_s, float* scale, const uint32_t* partial,
                       int n_partial, int8_t* xq, bool tiled, hipStream_t st)
{
    const RowOf ro = row_of(c_i >> 3);
    auto grid = [&](int u) {
        const int64_t n = (total + 256 * u - 1) / (256 * u);
        return dim3((unsigned)(n < 65536 ? n : 65536));  // (the kernel strides over the rest)
    };
    if (total >= ((int64_t)1 << 31)) sq_launch((quant_per_tensor_kernel<BF16, DYNAMIC, true, 2>), grid(2), dim3(256), 0, st, x, ldx, c_i, ro, total, inv_s, scale, partial, n_partial, xq, tiled);
    else if (total >= (DYNAMIC ? 1 << 19 : 1 << 21)) sq_launch((quant_per_tensor_kernel<BF16, DYNAMIC, false, 2>), grid(2), dim3(256), 0, st, x, ldx, c_i, ro, total, inv_s, scale, partial, n_partial, xq, tiled);
    else sq_launch((quant_per_tensor_kernel<BF16, DYNAMIC, false, 1>), grid(1), dim3(256), 0, st, x, ldx, c_i, ro, total, inv_s, scale, partial, n_partial, xq, tiled);
}

template <bool BF16, bool ATOMIC>
int launch_absmax(const uint16_t* x, int64_t ldx, int c_i, int64_t total, const float* inv_s, uint32_t* partial, hipStream_t st)
{
    constexpr int64_t chunk = (int64_t)kAbsmaxThreads * kAbsmaxUnroll;
    int64_t grid = (total + chunk - 1) / chunk;
    if (grid > kO2Parts) grid = kO2Parts;
    int64_t per = (total + grid - 1) / grid;
    per = (per + kAbsmaxThreads - 1) / kAbsmaxThreads * kAbsmaxThreads;  // (whole loads; in steps of a kilobyte the maxima are more, and by atomics 1000 x 9216 takes 17.9 us, so 16.8)
    grid = (total + per - 1) / per;
    const RowOf ro = row_of(c_i >> 3);
    if (total >= ((int64_t)1 << 31)) sq_launch((tensor_absmax_kernel<BF16, true, ATOMIC>), dim3((unsigned)grid), dim3(kAbsmaxThreads), 0, st, x, ldx, ro, total, per, inv_s, partial);
    else sq_launch((tensor_absmax_kernel<BF16, false, ATOMIC>), dim3((unsigned)grid), dim3(kAbsmaxThreads), 0, st, x, ldx, ro, total, per, inv_s, partial);
    return (int)grid;
}

// Tensors of one launch, by their 16-byte vectors: up to 2048 one workgroup (two vectors per thread), then one workgroup for each 1024.
constexpr int64_t kSmallVecs = 2048;
int64_t one_launch_vecs(bool smoothed) { return smoothed ? 4096 : 8192; }
template <bool BF16>
void launch_small(const uint16_t* x, int64_t ldx, int c_i, int64_t total, const float* inv_s, float* scale, int8_t* xq, bool tiled, hipStream_t st)
{
    const RowOf ro = row_of(c_i >> 3);
    if (total > kSmallVecs) sq_launch((quant_per_tensor_shared_kernel<BF16>), dim3((unsigned)((total + 1023) / 1024)), dim3(1024), 0, st, x, ldx, c_i, ro, (int)total, inv_s, scale, xq, tiled);
    else if (total > 1024) sq_launch((quant_per_tensor_small_kernel<BF16, 2>), dim3(1), dim3(1024), 0, st, x, ldx, c_i, ro, (int)total, inv_s, scale, xq, tiled);
    else sq_launch((quant_per_tensor_small_kernel<BF16, 1>), dim3(1), dim3(1024), 0, st, x, ldx, c_i, ro, (int)total, inv_s, scale, xq, tiled);
}

}  // namespace

extern "C" {

// Workspace of the per-tensor dynamic mode: the partial maxima.
size_t sq_quantize_workspace_bytes(void) { return kO2Parts * sizeof(uint32_t); }

sq_status sq_quantize_act(const void* x, sq_dtype dtype, int64_t t, int64_t c_i, int64_t ldx, const float* inv_s,
                          sq_act_mode mode, float* scale, int8_t* xq, sq_layout xq_layout, void* workspace,
                          size_t ws_bytes, void* stream)
{
    if (!x || !scale || !xq) return SQ_ERR_NULL;
    if (t <= 0 || c_i <= 0 || ldx < c_i || t >= ((int64_t)1 << 31) || c_i >= ((int64_t)1 << 31)) return SQ_ERR_SHAPE;
    if (dtype != SQ_F16 && dtype != SQ_BF16) return SQ_ERR_UNSUPPORTED;
    if (mode != SQ_PER_TOKEN_DYNAMIC && mode != SQ_PER_TENSOR_DYNAMIC && mode != SQ_PER_TENSOR_STATIC)
        return SQ_ERR_UNSUPPORTED;
    if (xq_layout != SQ_ROW_MAJOR && xq_layout != SQ_TILED) return SQ_ERR_UNSUPPORTED;
    if (xq_layout == SQ_TILED && (c_i & 63)) return SQ_ERR_ALIGN;
    const bool tiled = xq_layout == SQ_TILED;
    if ((c_i & 15) || (ldx & 7) || !sq_aligned16(x) || !sq_aligned16(xq) || (inv_s && !sq_aligned16(inv_s)))
        return SQ_ERR_ALIGN;
    if (mode == SQ_PER_TENSOR_DYNAMIC && (!workspace || ws_bytes < sizeof(uint32_t))) return SQ_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    const uint16_t* xp = (const uint16_t*)x;
    const bool bf = dtype == SQ_BF16;
    if (mode == SQ_PER_TOKEN_DYNAMIC) {
        if (bf) launch_per_token<true>(xp, ldx, (int)c_i, t, inv_s, scale, xq, tiled, st);
        else launch_per_token<false>(xp, ldx, (int)c_i, t, inv_s, scale, xq, tiled, st);
        return sq_launch_status();
    }
    const int64_t vecs = t * (c_i >> 3);
    if (mode == SQ_PER_TENSOR_DYNAMIC) {
        if (vecs <= one_launch_vecs(inv_s != nullptr)) {
            if (bf) launch_small<true>(xp, ldx, (int)c_i, vecs, inv_s, scale, xq, tiled, st);
            else launch_small<false>(xp, ldx, (int)c_i, vecs, inv_s, scale, xq, tiled, st);
            return sq_launch_status();
        }
        // Two launches: partial maxima, then every workgroup of the second kernel reduces them.  A caller with less than
        // the full workspace gets three (clear one cell, maxima by atomic, quantize); results are identical.
        if (reinterpret_cast<uintptr_t>(workspace) & 3u) return SQ_ERR_ALIGN;  // (words and atomics on words)
        int n_partial = 1;
        uint32_t* amax = (uint32_t*)workspace;
        if (ws_bytes >= sq_quantize_workspace_bytes()) {
            n_partial = bf ? launch_absmax<true, false>(xp, ldx, (int)c_i, vecs, inv_s, amax, st)
                           : launch_absmax<false, false>(xp, ldx, (int)c_i, vecs, inv_s, amax, st);
        } else {
            sq_launch(fill_u32_kernel, dim3(1), dim3(64), 0, st, amax, 0u, 1);
            if (bf) launch_absmax<true, true>(xp, ldx, (int)c_i, vecs, inv_s, amax, st);
            else launch_absmax<false, true>(xp, ldx, (int)c_i, vecs, inv_s, amax, st);
        }
        if (bf) launch_per_tensor<true, true>(xp, ldx, (int)c_i, vecs, inv_s, scale, amax, n_partial, xq, tiled, st);
        else launch_per_tensor<false, true>(xp, ldx, (int)c_i, vecs, inv_s, scale, amax, n_partial, xq, tiled, st);
    } else {
        if (bf) launch_per_tensor<true, false>(xp, ldx, (int)c_i, vecs, inv_s, scale, nullptr, 0, xq, tiled, st);
        else launch_per_tensor<false, false>(xp, ldx, (int)c_i, vecs, inv_s, scale, nullptr, 0, xq, tiled, st);
    }
    return sq_launch_status();
}

sq_status sq_act_absmax_per_channel(const void* x, sq_dtype dtype, int64_t t, int64_t c_i, float* out, void* stream)
{
    if (!x || !out) return SQ_ERR_NULL;
    if (t <= 0 || c_i <= 0 || t >= ((int64_t)1 << 31) || c_i >= ((int64_t)1 << 31)) return SQ_ERR_SHAPE;
    if (dtype != SQ_F16 && dtype != SQ_BF16) return SQ_ERR_UNSUPPORTED;
    if ((c_i & 15) || !sq_aligned16(x) || !sq_aligned16(out)) return SQ_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    // One row range while its 64-channel columns alone give every lane at most 16 rounds of loads, or while they fill the
    // chip; beyond that, ranges of 2048 rows and more, about four workgroups per compute unit.  (Narrow batches too: the twelve
    // workgroups of 2048 x 768 take 6.7 us, 256 of them with an atomic per channel took 43; 512 x 768 3.6 / 42.)
    const int64_t cols = (c_i + 63) / 64;
    int64_t ranges = (t + 2047) / 2048;
    if (ranges > (1024 + cols - 1) / cols) ranges = (1024 + cols - 1) / cols;
    const int64_t per = (t + ranges - 1) / ranges;
    ranges = (t + per - 1) / per;
    if (ranges > 1) sq_launch(fill_u32_kernel, dim3((unsigned)((c_i + 255) / 256)), dim3(256), 0, st, (uint32_t*)out, 0u, (int)c_i);
    constexpr int64_t most = 1 << 23;  // columns per launch: a grid stays below 2^32 threads
    for (int64_t first = 0; first < cols; first += most) {
        const dim3 grid((unsigned)(cols - first < most ? cols - first : most), (unsigned)ranges);
        if (dtype == SQ_BF16) sq_launch(act_absmax_per_channel_kernel<true>, grid, dim3(256), 0, st, (const uint16_t*)x, (int)c_i, t, per, (uint32_t*)out, (int)first);
        else sq_launch(act_absmax_per_channel_kernel<false>, grid, dim3(256), 0, st, (const uint16_t*)x, (int)c_i, t, per, (uint32_t*)out, (int)first);
    }
    return sq_launch_status();
}

}  // extern "C"
