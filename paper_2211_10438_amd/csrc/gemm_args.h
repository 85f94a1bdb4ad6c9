// Argument block and epilogue arithmetic shared by the INT8 GEMM kernels (gfx950).
#pragma once
#include "common.h"

#define GPTR(p) ((const __attribute__((address_space(1))) void*)(p))
#define LPTR(p) ((__attribute__((address_space(3))) void*)(p))

struct GemmArgs {
    const int8_t* A;  // [batch][M, K], row stride lda bytes
    const int8_t* B;  // [batch][N, K], row stride ldb bytes
    int M, N, K;
    int64_t lda, ldb;
    int64_t strideA, strideB, strideC;  // batch strides in elements
    int tiles_m, tiles_n, splits, iters_per_split;
    // dequant epilogue
    void* C;  // [batch][M, N] 16-bit, row stride N
    const float* x_scale;  // [M] or [1] or NULL (then `alpha` is the whole scale)
    int per_token;
    const float* w_scale;  // [1], or [N] with w_per_channel
    int w_per_channel;
    float alpha;
    const float* bias;     // [N] or NULL
    const void* residual;  // [M, N] out dtype or NULL
    int relu;
    // int32 output (raw accumulators or split-K partials): [splits][M, N]
    int32_t* acc_out;
    // int8 output (producer-side fusion): when q8_step is set, the 16-bit value the epilogue would have stored is
    // quantized with the calibrated step q8_step[0] (Eq. 1, static) and written to q8_out [M, N] instead of C.
    const float* q8_step;
    int8_t* q8_out;
    int q8_tiled;
};

// Static per-tensor quantization of a value that has already been rounded to the 16-bit type `BF16` selects:
// the same arithmetic as the static mode of the activation quantizer (x * fl32(1 / Delta), nearest-even, +-127).
template <bool BF16> SQ_DEVICE int requant_code(uint32_t bits16, float r)
{
    return round_code(load16_bits<BF16>(bits16) * r);
}

template <int N> SQ_DEVICE void wait_vmcnt_imm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// 16 bytes per lane from a buffer into LDS (lane l to dst + 16 l); what lies outside the buffer arrives as zeros and costs no traffic.
template <bool NT> SQ_DEVICE void buffer_to_lds(__amdgpu_buffer_rsrc_t r, char* dst, uint32_t lane_offset, int offset)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, LPTR(dst), 16, (int)lane_offset, offset, 0, NT ? 2 : 0);
}

// Byte-transposing LDS reads (16 lanes name the 8-byte halves of eight rows' 16 bytes; lane i receives byte i of each row), and the wait for
// them: out[2 k], out[2 k + 1] from the LDS addresses p[k] + LO and p[k] + HI.  In asm because the compiler, before the builtin, waits for
// every global->LDS load in flight -- those of the next stages, which nobody needs yet -- as if they wrote what is read here.  (It
// sees neither these reads nor the loads they follow: the caller's barriers order them.)
template <int LO, int HI, int N> SQ_DEVICE void lds_read_tr(const uint32_t (&p)[N], v2i (&out)[2 * N])
{
    static_assert(N >= 1 && N <= 4, "columns blocks at a time");
    if constexpr (N == 1) {
        asm volatile("ds_read_b64_tr_b8 %0, %2 offset:%3\n\t" "ds_read_b64_tr_b8 %1, %2 offset:%4\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(out[0]), "=&v"(out[1])
                 : "v"(p[0]), "n"(LO), "n"(HI));
    } else if constexpr (N == 2) {
        asm volatile("ds_read_b64_tr_b8 %0, %4 offset:%6\n\t" "ds_read_b64_tr_b8 %1, %4 offset:%7\n\t"
                 "ds_read_b64_tr_b8 %2, %5 offset:%6\n\t" "ds_read_b64_tr_b8 %3, %5 offset:%7\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(out[0]), "=&v"(out[1]), "=&v"(out[2]), "=&v"(out[3])
                 : "v"(p[0]), "v"(p[1]), "n"(LO), "n"(HI));
    } else if constexpr (N == 3) {
        asm volatile("ds_read_b64_tr_b8 %0, %6 offset:%9\n\t" "ds_read_b64_tr_b8 %1, %6 offset:%10\n\t"
                 "ds_read_b64_tr_b8 %2, %7 offset:%9\n\t" "ds_read_b64_tr_b8 %3, %7 offset:%10\n\t"
                 "ds_read_b64_tr_b8 %4, %8 offset:%9\n\t" "ds_read_b64_tr_b8 %5, %8 offset:%10\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(out[0]), "=&v"(out[1]), "=&v"(out[2]), "=&v"(out[3]), "=&v"(out[4]), "=&v"(out[5])
                 : "v"(p[0]), "v"(p[1]), "v"(p[2]), "n"(LO), "n"(HI));
    } else {
        asm volatile("ds_read_b64_tr_b8 %0, %8 offset:%12\n\t" "ds_read_b64_tr_b8 %1, %8 offset:%13\n\t"
                 "ds_read_b64_tr_b8 %2, %9 offset:%12\n\t" "ds_read_b64_tr_b8 %3, %9 offset:%13\n\t"
                 "ds_read_b64_tr_b8 %4, %10 offset:%12\n\t" "ds_read_b64_tr_b8 %5, %10 offset:%13\n\t"
                 "ds_read_b64_tr_b8 %6, %11 offset:%12\n\t" "ds_read_b64_tr_b8 %7, %11 offset:%13\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(out[0]), "=&v"(out[1]), "=&v"(out[2]), "=&v"(out[3]), "=&v"(out[4]), "=&v"(out[5]), "=&v"(out[6]), "=&v"(out[7])
                 : "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3]), "n"(LO), "n"(HI));
    }
}
SQ_DEVICE uint32_t lds_address(const char* p) { return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)p; }

// Outer-dimension scaling of Eq. 2 on one accumulator: (float)acc * c, then the optional terms in the
// order bias, ReLU, residual, then one rounding to the 16-bit output type.
template <bool BF16>
SQ_DEVICE uint32_t dequant_one(int acc, float c, float bias, bool has_bias, bool relu, uint32_t res_bits, bool has_res)
{
    float v = (float)acc * c;
    if (has_bias) v = v + bias;
    if (relu) v = v > 0.0f ? v : 0.0f;
    if (has_res) v = v + load16_bits<BF16>(res_bits);
    return store16_bits<BF16>(v);
}

// The same for two neighbouring outputs, narrowed together (lo = first): one conversion instruction for the pair.
// (the accumulators arrive already converted to fp32: exact up to 2^24, round-to-nearest-even beyond, like the cast)
template <bool BF16>
SQ_DEVICE uint32_t dequant_pair_f(float acc0, float acc1, float c0, float c1, float bias0, float bias1, bool has_bias, bool relu,
                                  uint32_t res_pair, bool has_res)
{
    float v0 = acc0 * c0, v1 = acc1 * c1;
    if (has_bias) { v0 = v0 + bias0; v1 = v1 + bias1; }
    if (relu) { v0 = v0 > 0.0f ? v0 : 0.0f; v1 = v1 > 0.0f ? v1 : 0.0f; }
    if (has_res) { v0 = v0 + load16_bits<BF16>(res_pair); v1 = v1 + load16_bits<BF16>(res_pair >> 16); }
    return store16x2_bits<BF16>(v0, v1);
}
template <bool BF16>
SQ_DEVICE uint32_t dequant_pair(int acc0, int acc1, float c0, float c1, float bias0, float bias1, bool has_bias, bool relu,
                                uint32_t res_pair, bool has_res)
{
    return dequant_pair_f<BF16>((float)acc0, (float)acc1, c0, c1, bias0, bias1, has_bias, relu, res_pair, has_res);
}

// Weight-streaming GEMM for few-token shapes (gemm_i8_stream.hip).  No plan: the shape is left to the tile kernels.  Without a K split
// (gk = 1) the kernel writes the final output itself; with one it writes int32 partial sums to a.acc_out[gk][M][N] (which the
// caller points at a workspace) and the split-K reduction kernel finishes the job.
struct StreamArgs {
    int gn;          // slabs (workgroups along C_o)
    int gk;          // K splits (workgroups along K); > 1: int32 partials go to acc_out[gk][M][N]
    int units;       // 16-column units of N
    int na;          // 16-row blocks of A
    int ksub;        // 64-byte K steps per stage
    int iters;       // stages per workgroup: K / 64 / gk / ksub
    int nt_w;        // weight loads carry the non-temporal hint
    int regs;        // the register-direct kernel runs this plan
    int tiled, to_i32, bf16;
    double us;       // modelled time of the plan
};
bool sq_stream_gemm_plan(int64_t M, int64_t N, int64_t K, int64_t batch, bool tiled, StreamArgs* out);
bool sq_stream_rows_plan(int64_t M, int64_t N, int64_t K, StreamArgs* out);
void sq_stream_gemm_launch(const GemmArgs& a, StreamArgs q, bool to_i32, bool bf16, bool tiled, hipStream_t st);

// Strip kernel for attention scores (bmm_strip.hip): B = [N, K] with K <= 128, alpha-only epilogue.
bool sq_strip_bmm_eligible(int64_t M, int64_t N, int64_t K, int64_t batch);
void sq_strip_bmm_launch(const GemmArgs& a, int batch, bool bf16, hipStream_t st);

// P V of attention (bmm_pv.hip): B = [K, N], N % 16 == 0, alpha-only epilogue.
void sq_pv_bmm_launch(GemmArgs a, int batch, bool bf16, hipStream_t st);

// Few output tiles for the chip (gemm_direct.h): 16 mb tokens x 16 nb channels per workgroup of nw waves, one kernel, no workspace.
// False: no such instantiation, or more workgroups than a launch holds.
struct DirectArgs {
    int tiles_m, tiles_n;
    int n_outer;  // the tiles are walked token tiles first (1: those of one channel tile side by side) or channel tiles first (0)
    int to_i32, bf16;
};
struct DirectPlan {
    int mb, nb, nw;  // 0: none
    double us;       // modelled time
};
DirectPlan sq_direct_gemm_plan(int64_t M, int64_t N, int64_t K, bool tiled);
bool sq_direct_gemm_launch(const GemmArgs& a, int mb, int nb, int nw, bool to_i32, bool bf16, bool tiled, hipStream_t st);
bool sq_direct_gemm_launch_tiled(const GemmArgs& a, const DirectArgs& q, int mb, int nb, int nw, hipStream_t st);
bool sq_direct_gemm_launch_rows(const GemmArgs& a, const DirectArgs& q, int mb, int nb, int nw, hipStream_t st);
