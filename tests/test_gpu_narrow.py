"""Layers of few tokens and few output channels, which the direct kernel takes: ragged tokens and channels, 64-byte K steps dealt in pairs
to the waves, a last step of one to three 16-byte chunks; and K splits of the tile kernels.  Against the exact integer product and the
fixed fp32 epilogue in torch: outputs identical."""
import pytest
import torch

from paper_2211_10438_amd import binding as sq
from tests._util import tiled_index

pytestmark = pytest.mark.gpu

# (tokens, C_i, C_o); odd C_o, C_o off 16 and off 4, one K step, an odd number of steps, fewer pairs of steps than waves, a
# K tail (row-major only)
CASES = [(1, 16, 1), (2, 64, 8), (15, 128, 24), (16, 768, 3072), (17, 192, 100), (24, 1024, 772), (32, 1024, 772), (33, 1088, 16), (64, 960, 2048),
         (65, 80, 333), (100, 784, 768), (128, 1008, 1030), (128, 3072, 512), (1, 5120, 4095), (4, 12288, 2304), (3, 2064, 3000),
         # wider than one 16-channel unit per compute unit: up to 16 tokens without a workspace, then (17 tokens) by the planner's models
         (4, 2048, 5120), (16, 1088, 4112), (9, 512, 6544), (17, 1024, 5120)]


def _tile(codes):
    rows, k = codes.shape
    buf = sq.empty_codes(rows, k, sq.TILED)
    flat = (buf._base if buf._base is not None else buf).reshape(-1)
    flat.fill_(77)  # the padding rows hold something
    flat[torch.from_numpy(tiled_index(rows, k)).cuda()] = codes
    return buf


@pytest.mark.parametrize("t,c_i,c_o", CASES)
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("kind", ["plain", "all", "per_channel_q8", "i32"])
def test_narrow_linear(t, c_i, c_o, dtype, kind):
    print(f"narrow {t}x{c_i}->{c_o} {dtype} {kind}", flush=True)
    if (t, c_i, c_o) in CASES[:-1]:
        assert any(sq.lib().sq_probe_narrow_gemm(t, c_i, c_o, layout) for layout in [sq.ROW_MAJOR] + ([sq.TILED] if c_i % 64 == 0 else []))
    g = torch.Generator(device="cuda").manual_seed(t + c_i + c_o)
    x, w = (torch.randint(-127, 128, s, generator=g, device="cuda", dtype=torch.int32).to(torch.int8) for s in ((t, c_i), (c_o, c_i)))
    xs = torch.rand(t, generator=g, device="cuda") * 0.01 + 0.001
    full = kind == "all"
    per_channel = kind == "per_channel_q8"
    ws = (torch.rand(c_o, generator=g, device="cuda") * 0.001 + 1e-4) if per_channel else torch.full((1,), 3e-4, device="cuda")
    bias = torch.randn(c_o, generator=g, device="cuda") if full or per_channel else None
    res = torch.randn((t, c_o), generator=g, device="cuda").to(dtype) if full else None
    acc = (x.double() @ w.double().t()).to(torch.int32)
    v = acc.float() * (xs[:, None] * ws)
    if bias is not None:
        v = v + bias
    if full:
        v = v.clamp_min(0) + res.float()
    v16 = v.to(dtype)
    for layout in [sq.ROW_MAJOR] + ([sq.TILED] if c_i % 64 == 0 else []):
        xq, wq = (x, w) if layout == sq.ROW_MAJOR else (_tile(x), _tile(w))
        if kind == "i32":
            assert torch.equal(sq.i8_gemm_i32(xq, wq, layout=layout), acc)
        elif per_channel:
            if c_o % 8:
                continue
            step = torch.full((1,), 0.037, device="cuda")
            r = (torch.ones(1) / torch.full((1,), 0.037)).cuda()  # one IEEE division
            codes = sq.w8a8_linear_q8(xq, xs, wq, ws, step, dtype, bias=bias, layout=layout)
            assert torch.equal(codes, (v16.float() * r).round().clamp(-127, 127).to(torch.int8))
        else:
            y = sq.w8a8_linear(xq, xs, wq, ws, dtype, bias=bias, residual=res, relu=full, layout=layout)
            assert torch.equal(y.view(torch.int16), v16.view(torch.int16))


# K splits of the tile kernels and their reduction, one column per thread and (C_o % 4 == 0, from 2^17 outputs on) four
@pytest.mark.parametrize("t,c_i,c_o", [(79, 20928, 1656), (79, 20928, 1696), (4, 15808, 8), (150, 12160, 2497), (212, 13312, 1641), (141, 18240, 1648),
                                         (135, 9344, 5528)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_split_reduction(t, c_i, c_o, dtype):
    print(f"split reduction {t}x{c_i}->{c_o} {dtype}", flush=True)
    plans = [sq.probe_linear_plan(t, c_i, c_o, layout) for layout in (sq.ROW_MAJOR, sq.TILED)]
    assert any(p[0] == 2 and p[2] > 1 for p in plans), plans
    for kind in ("plain", "all", "i32") + (("per_channel_q8",) if c_o % 8 == 0 else ()):
        test_narrow_linear(t, c_i, c_o, dtype, kind)
