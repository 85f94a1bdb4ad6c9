"""GPU parity of the linear layer whose epilogue applies the next kernel's static activation quantizer
(sq_w8a8_linear_q8).  The expected codes are the oracle's own chain: w8a8_linear (16-bit output) followed by
quantize_act in static mode -- the fused kernel must produce exactly those codes, on every GEMM path."""
import numpy as np
import pytest
import torch

import oracle
from paper_2211_10438_amd import binding as sq
from paper_2211_10438_amd import synth
from tests._util import (BF16, F16, dev, random_bf16_bits, rows_to_tiled_dev, tiled_index, tiled_to_rows, to_dev_16, torch_dtype)
from tests.test_gpu_narrow import _tile

pytestmark = pytest.mark.gpu


def _progress(msg):
    print(f"[case] {msg}", flush=True)


CASES = [
    # t, c_i, c_o, mid dtype, bias, relu, residual, in layout, out layout, per-channel W
    (300, 1024, 1000, BF16, True, True, False, sq.ROW_MAJOR, sq.ROW_MAJOR, False),   # direct kernel, ragged
    (2048, 256, 1536, F16, False, True, False, sq.TILED, sq.TILED, False),           # FC1 + ReLU -> codes for FC2
    (513, 320, 2048, F16, True, False, True, sq.ROW_MAJOR, sq.TILED, True),          # K tail, residual, per-channel W
    (16, 4096, 1024, BF16, True, False, False, sq.TILED, sq.ROW_MAJOR, False),       # direct kernel, few channels
    (5, 1024, 4096, F16, True, True, True, sq.ROW_MAJOR, sq.TILED, False),           # direct kernel, five tokens
    (128, 4096, 4096, BF16, True, False, False, sq.TILED, sq.TILED, True),           # direct kernel, 128 tokens
    (70, 1088, 8192, F16, False, False, False, sq.TILED, sq.ROW_MAJOR, False),       # direct kernel, 70 tokens
    (124, 20480, 1088, F16, True, True, False, sq.TILED, sq.TILED, True),            # split-K tiles + reduction kernel
    (79, 20928, 1696, BF16, True, False, True, sq.ROW_MAJOR, sq.ROW_MAJOR, False),   # the same, row-major
    (5, 768, 16512, F16, True, True, True, sq.ROW_MAJOR, sq.TILED, False),           # weight streaming
    (64, 8320, 4160, BF16, True, False, False, sq.TILED, sq.TILED, True),            # streaming with a K split
    (64, 1216, 8640, F16, False, False, False, sq.TILED, sq.ROW_MAJOR, False),       # streaming straight into registers
]
PLANNED = {(2048, 256): 2, (124, 20480): 2, (79, 20928): 2, (5, 768): 1, (64, 8320): 1, (64, 1216): 1}  # the others: direct kernel


@pytest.mark.parametrize("t,c_i,c_o,mid,use_bias,relu,use_res,lay_in,lay_out,w_pc", CASES)
def test_linear_q8_matches_linear_then_static_quantize(t, c_i, c_o, mid, use_bias, relu, use_res, lay_in, lay_out, w_pc):
    _progress(f"linear_q8 t={t} c_i={c_i} c_o={c_o} mid={mid} in={lay_in} out={lay_out} w_pc={w_pc}")
    assert sq.probe_linear_plan(t, c_i, c_o, lay_in)[0] == PLANNED.get((t, c_i), 0)
    seed = 11000 + t + c_i + c_o
    case = synth.linear_case(t, c_i, c_o, 0.01, 40.0, seed, calib_tokens=64)
    ax = oracle.act_absmax_per_channel(case["x_calib"], F16)
    aw = oracle.weight_absmax_per_in_channel(case["w"], F16)
    s, inv_s = oracle.smooth_scales(ax, aw, 0.5)
    wq, ws = oracle.prepare_weight(case["w"], F16, s, per_channel=w_pc)
    xq, xs = oracle.quantize_act(case["x"], F16, oracle.PER_TOKEN_DYNAMIC, inv_s=inv_s)
    bias = synth.bias(c_o, seed + 9) if use_bias else None
    res = None
    if use_res:
        res = synth.normal_fp16((t, c_o), seed + 10) if mid == F16 else random_bf16_bits((t, c_o), seed + 10)
    y16 = oracle.w8a8_linear(xq, xs, wq, ws, mid, bias=bias, residual_bits=res, relu=relu, w_per_channel=w_pc)
    # calibrated output step: a little below absmax / 127 so that the saturation to +-127 is exercised as well
    amax = np.abs(oracle.f32_from_bits16(y16, mid)).max()
    step = np.float32(0.9) * np.float32(amax) / np.float32(127.0)
    ref, _ = oracle.quantize_act(y16, mid, oracle.PER_TENSOR_STATIC, static_scale=step)
    assert np.abs(ref).max() == 127
    xq_d, wq_d = (rows_to_tiled_dev(xq), rows_to_tiled_dev(wq)) if lay_in == sq.TILED else (dev(xq), dev(wq))
    yq = sq.w8a8_linear_q8(xq_d, dev(xs), wq_d, dev(ws), dev(np.array([step], np.float32)), torch_dtype(mid),
                           bias=None if bias is None else dev(bias), residual=None if res is None else to_dev_16(res, mid),
                           relu=relu, layout=lay_in, out_layout=lay_out)
    got = tiled_to_rows(yq) if lay_out == sq.TILED else yq.cpu().numpy()
    bad = np.argwhere(got != ref)
    assert bad.size == 0, f"{len(bad)} codes differ, first at {bad[:5].tolist()}"


def test_linear_q8_zero_step_gives_zero_codes():
    _progress("linear_q8 zero step")
    xq, wq = synth.int8_codes((40, 256), 1), synth.int8_codes((512, 256), 2)
    yq = sq.w8a8_linear_q8(dev(xq), dev(np.full(40, 1e-4, np.float32)), dev(wq), dev(np.ones(1, np.float32)),  # finite values
                           dev(np.zeros(1, np.float32)), torch_dtype(F16))
    assert not yq.cpu().numpy().any()


# Every tile, unsplit, with c_o of whole 64 (both output layouts), of 16 and of 8; both MFMA forms of the wide ones (c_i a multiple of 128 or not).
TILE_FORMS = [
    (175, 128, 12160, sq.ROW_MAJOR, 128128), (2091, 128, 1232, sq.TILED, 128128), (162, 64, 12488, sq.TILED, 128128),
    (114, 464, 20672, sq.ROW_MAJOR, 128256), (119, 432, 19792, sq.ROW_MAJOR, 128256), (119, 496, 18920, sq.ROW_MAJOR, 128256),
    (315, 320, 18112, sq.TILED, 192160), (281, 336, 16848, sq.ROW_MAJOR, 192160), (315, 320, 18152, sq.TILED, 192160),
    (522, 320, 17408, sq.TILED, 192224), (566, 320, 17760, sq.ROW_MAJOR, 192224), (519, 384, 18584, sq.TILED, 192224),
    (197, 320, 11328, sq.TILED, 256128), (137, 288, 17328, sq.ROW_MAJOR, 256128), (135, 304, 20376, sq.ROW_MAJOR, 256128),
    (773, 464, 8704, sq.ROW_MAJOR, 256160), (824, 320, 17104, sq.TILED, 256160), (803, 448, 8520, sq.ROW_MAJOR, 256160),
    (541, 384, 14272, sq.ROW_MAJOR, 256192), (391, 320, 18368, sq.TILED, 256192), (775, 384, 8208, sq.TILED, 256192), (389, 272, 17944, sq.ROW_MAJOR, 256192),
    (643, 384, 16832, sq.TILED, 256256), (612, 272, 16640, sq.ROW_MAJOR, 256256), (592, 320, 16720, sq.TILED, 256256), (795, 384, 13176, sq.TILED, 256256),
    (1373, 768, 14592, sq.TILED, 256384), (1406, 272, 13760, sq.ROW_MAJOR, 256384), (1166, 768, 16480, sq.TILED, 256384), (1125, 288, 17240, sq.ROW_MAJOR, 256384)]


@pytest.mark.parametrize("t,c_i,c_o,layout,tile", TILE_FORMS)
def test_linear_q8_of_every_tile(t, c_i, c_o, layout, tile):
    """Codes of the fused call against those of the 16-bit call's values, by the static quantizer's formula: identical."""
    assert sq.lib().sq_probe_linear_tile(t, c_i, c_o, layout) == 1000000 + tile
    g = torch.Generator(device="cuda").manual_seed(t + c_o)
    rows = [torch.randint(-127, 128, s, generator=g, device="cuda", dtype=torch.int32).to(torch.int8) for s in ((t, c_i), (c_o, c_i))]
    xq, wq = [_tile(a) for a in rows] if layout == sq.TILED else rows
    xs, ws, bias = (torch.rand(n, generator=g, device="cuda") * 0.01 + 0.001 for n in (t, c_o, c_o))
    for dtype in (torch.float16, torch.bfloat16):
        res = torch.randn(t, c_o, generator=g, device="cuda").to(dtype)
        for kw in (dict(), dict(bias=bias, residual=res, relu=True)):
            _progress(f"tile {tile} q8 {t}x{c_i}->{c_o} layout {layout} {dtype} {list(kw)}")
            y = sq.w8a8_linear(xq, xs, wq, ws, dtype, layout=layout, **kw)
            step = (0.8 * y.float().abs().amax() / 127).reshape(1)
            want = (y.float() * (1.0 / step)).round().clamp(-127, 127).to(torch.int8)
            assert want.abs().max() == 127
            for out_layout in (sq.ROW_MAJOR, sq.TILED)[: 2 if c_o % 64 == 0 else 1]:
                got = sq.w8a8_linear_q8(xq, xs, wq, ws, step, dtype, layout=layout, out_layout=out_layout, **kw)
                if out_layout == sq.TILED:  # (the padding rows of the last block are undefined)
                    got = (got._base if got._base is not None else got).reshape(-1)[torch.from_numpy(tiled_index(t, c_o)).cuda()]
                assert torch.equal(got, want)
