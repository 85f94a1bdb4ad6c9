/*
 * sqmi -- measurement aids of the library, NOT part of the method's boundary (that is sqmi.h).
 * bench.py uses them to report kernels against what the hardware sustains, the tests to reach a kernel whatever the
 * library's choice of kernel for a shape is.
 */
#ifndef SQMI_PROBE_H
#define SQMI_PROBE_H

#include "sqmi.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Runs `iters` rounds of 16 register-fed INT8 MFMAs (16x16x64, the shape of the compute-bound GEMM tiles) on each of
 * the 8 waves of `workgroups` workgroups, i.e. workgroups * 8 * iters * 16 * 32768 integer operations, with no
 * memory traffic inside the loop.  The operand registers are filled once from `data` (device int8, at least
 * workgroups * 49152 bytes: the bit patterns matter, the sustained clock depends on them); sink: device int32
 * [workgroups * 512], overwritten.  bench.py times it to report the GEMM against what the matrix pipes sustain. */
sq_status sq_probe_mfma_i8(const int8_t* data, size_t data_bytes, int workgroups, int iters, int32_t* sink, void* stream);

/* The form of the fused attention kernel that sq_w8a8_attention (causal != 0: sq_w8a8_attention_causal) takes for these
 * sizes: 1 = row blocks of 128 queries, 2 = few queries (blocks of 16); 0 for sizes it refuses.  No GPU work. */
int sq_probe_attention_form(int64_t b, int64_t s_q, int64_t s_k, int64_t d, int causal);

/* The row block (of 128 queries) that workgroup `block` of the row-block form works on under the causal mask, its head in
 * *head; below 0 past the launch's last workgroup.  Workgroups go round-robin to the 8 XCDs.  No GPU work. */
int sq_probe_attention_place(int64_t block, int64_t b, int64_t s_q, int64_t s_k, int64_t d, int64_t* head);

/* sq_w8a8_attention / _causal in the form named (1 or 2, else SQ_ERR_UNSUPPORTED; 2 also where that form cannot hold the
 * scores, s_k > 8192).  Other arguments, checks and results are theirs. */
sq_status sq_probe_attention(int form, int causal, const int8_t* q, const int8_t* k, const int8_t* v, float alpha1,
                             float alpha2, void* o, sq_dtype out, int64_t b, int64_t s_q, int64_t s_k, int64_t d,
                             int64_t stride_q, int64_t stride_k, int64_t stride_v, int64_t stride_o, int8_t* p_codes,
                             void* stream);

/* 1 where a linear layer of this size counts as one of few tokens and few output channels (direct kernel, never a workspace), else 0.
 * No GPU work. */
int sq_probe_narrow_gemm(int64_t t, int64_t c_i, int64_t c_o, sq_layout layout);

/* sq_w8a8_linear by the direct kernel (operands from memory into MFMA registers, K dealt to the waves of a workgroup) with tiles of
 * 16 mb tokens x 16 nb channels and nw waves, whatever the library would choose; SQ_ERR_UNSUPPORTED where that combination is not
 * built or its launch would be too large.  Other arguments, checks and results are those of sq_w8a8_linear. */
sq_status sq_probe_linear_blocks(int mb, int nb, int nw, const int8_t* xq, const float* x_scale, int x_scale_per_token, const int8_t* wq,
                                 const float* w_scale, int w_scale_per_channel, const float* bias, const void* residual, int relu,
                                 void* y, sq_dtype out, int64_t t, int64_t c_i, int64_t c_o, sq_layout layout, void* stream);

/* 100 mb + 10 nb + nw where a linear layer of this size runs the direct kernel, 0 where it runs another.  No GPU work. */
int sq_probe_linear_form(int64_t t, int64_t c_i, int64_t c_o, sq_layout layout);

/* 1000000 s + 1000 m + n where it runs m x n tiles staged through LDS with s K splits, else 0.  No GPU work. */
int sq_probe_linear_tile(int64_t t, int64_t c_i, int64_t c_o, sq_layout layout);

/* The plan of a linear layer of this size: out[0] the kernel (0 direct, 1 weight streaming, 2 tiles staged through LDS), out[1] its variant
 * (direct: 100 mb + 10 nb + nw; streaming: 1 the register-direct kernel, 0 the LDS ring; tiles: their number in the library), out[2] the K
 * splits, out[3] the 64-byte K steps of a split, out[4] and out[5] streaming: slabs and 16-channel units, tiles: token and channel tiles,
 * direct: 0.  No GPU work. */
sq_status sq_probe_linear_plan(int64_t t, int64_t c_i, int64_t c_o, sq_layout layout, int64_t out[6]);

#ifdef __cplusplus
}
#endif
#endif /* SQMI_PROBE_H */
