"""The weight-streaming kernel for 33 to 128 tokens (tiled): three to eight token blocks, slabs whose units do not divide among the three
unit groups, with a shorter last slab, odd numbers of stages, K splits.  Against the exact integer product: outputs identical."""
import pytest
import torch

from paper_2211_10438_amd import binding as sq
from tests.test_gpu_narrow import _tile

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("t,c_i,c_o", [(40, 1024, 16441), (48, 2368, 24908), (70, 2624, 20562), (81, 5760, 17240), (100, 3008, 24765), (112, 1280, 16471),
                                       (113, 1728, 8332), (128, 1664, 28728), (100, 2368, 45144), (120, 2880, 10936), (96, 2688, 16528), (128, 1216, 40976),
                                       (49, 6912, 4312), (65, 5504, 16981), (101, 7488, 8209)])
def test_units_and_blocks(t, c_i, c_o):
    assert sq.probe_linear_plan(t, c_i, c_o, sq.TILED)[:2] == (1, 1)
    print(f"stream {t}x{c_i}->{c_o}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(t + c_i + c_o)
    x, w = (torch.randint(-127, 128, s, generator=g, device="cuda", dtype=torch.int32).to(torch.int8) for s in ((t, c_i), (c_o, c_i)))
    xs, ws = torch.rand(t, generator=g, device="cuda") * 0.01 + 0.001, torch.rand(c_o, generator=g, device="cuda") * 0.001 + 1e-4
    bias = torch.randn(c_o, generator=g, device="cuda")
    acc = (x.double() @ w.double().t()).to(torch.int32)
    xq, wq = _tile(x), _tile(w)
    assert torch.equal(sq.i8_gemm_i32(xq, wq, layout=sq.TILED), acc)
    for dtype in (torch.float16, torch.bfloat16):
        y = sq.w8a8_linear(xq, xs, wq, ws, dtype, bias=bias, layout=sq.TILED)
        assert torch.equal(y.view(torch.int16), (acc.float() * (xs[:, None] * ws) + bias).to(dtype).view(torch.int16))


@pytest.mark.parametrize("t,c_i,c_o", [(33, 3584, 10009), (48, 2624, 20012), (70, 4032, 24563), (81, 2048, 16392), (100, 4160, 27648), (112, 2432, 12289),
                                       (113, 3008, 30011), (128, 4096, 12288), (120, 1728, 22264), (62, 1984, 14120), (36, 2240, 40984)])
def test_row_major_units_and_blocks(t, c_i, c_o):
    """The same kernel on row-major operands: rows of the last unit and the last token block that are not there, steps in pairs (odd
    numbers of steps and of pairs), every output type."""
    assert sq.probe_linear_plan(t, c_i, c_o, sq.ROW_MAJOR)[:3] == (1, 1, 1)
    print(f"stream rows {t}x{c_i}->{c_o}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(t + c_i + c_o)
    x, w = (torch.randint(-127, 128, s, generator=g, device="cuda", dtype=torch.int32).to(torch.int8) for s in ((t, c_i), (c_o, c_i)))
    xs, ws = torch.rand(t, generator=g, device="cuda") * 0.01 + 0.001, torch.rand(c_o, generator=g, device="cuda") * 0.001 + 1e-4
    bias = torch.randn(c_o, generator=g, device="cuda")
    acc = (x.double() @ w.double().t()).to(torch.int32)
    assert torch.equal(sq.i8_gemm_i32(x, w), acc)
    for dtype in (torch.float16, torch.bfloat16):
        res = torch.randn((t, c_o), generator=g, device="cuda").to(dtype)
        v = ((acc.float() * (xs[:, None] * ws) + bias).clamp_min(0) + res.float()).to(dtype)
        y = sq.w8a8_linear(x, xs, w, ws, dtype, bias=bias, relu=True, residual=res)
        assert torch.equal(y.view(torch.int16), v.view(torch.int16))
        if c_o % 8 == 0:
            step = torch.full((1,), 0.037, device="cuda")
            r = (torch.ones(1) / torch.full((1,), 0.037)).cuda()
            q = sq.w8a8_linear_q8(x, xs, w, ws, step, dtype, bias=bias, relu=True, residual=res)
            assert torch.equal(q, (v.float() * r).round().clamp(-127, 127).to(torch.int8))


@pytest.mark.parametrize("m,k,n", [(48, 2624, 20012), (112, 2432, 12289), (100, 4160, 27648), (36, 2240, 40984)])
def test_one_batch_product_with_alpha_alone(m, k, n):
    """The same kernel as sq_w8a8_bmm of one batch entry reaches it: no scales, no bias, alpha in their place."""
    assert sq.probe_linear_plan(m, k, n, sq.ROW_MAJOR)[:3] == (1, 1, 1)
    print(f"stream rows, alpha alone {m}x{k}->{n}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(m + k + n)
    a, b = (torch.randint(-127, 128, s, generator=g, device="cuda", dtype=torch.int32).to(torch.int8) for s in ((1, m, k), (1, n, k)))
    acc = (a[0].double() @ b[0].double().t()).float()
    for dtype in (torch.float16, torch.bfloat16):
        c = sq.w8a8_bmm(a, b, True, 3e-4, dtype)
        v = (acc * torch.tensor(3e-4, dtype=torch.float32, device="cuda")).to(dtype)
        assert torch.equal(c[0].view(torch.int16), v.view(torch.int16))
