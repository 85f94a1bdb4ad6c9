"""Tiles whose output rows are not whole 16-byte pieces (C_o a multiple of 4, of 2, odd): every tile, both MFMA forms of the wide ones, with and
without a residual, the residual in the output's place too.  Against the exact integer product and the fixed fp32 epilogue: identical, and nothing
outside the output is written."""
import pytest
import torch

from paper_2211_10438_amd import binding as sq
from tests.test_gpu_narrow import _tile

pytestmark = pytest.mark.gpu
R, T = sq.ROW_MAJOR, sq.TILED
GUARD = 1 << 15  # values

SHAPES = [
    (343, 64, 17220, T, 128128), (346, 64, 16434, R, 128128), (339, 64, 16777, R, 128128),
    (289, 592, 16532, R, 192160), (346, 528, 17802, R, 192160), (351, 528, 16761, R, 192160),
    (575, 384, 16780, R, 192224), (541, 480, 16634, R, 192224), (537, 480, 16753, R, 192224),
    (140, 992, 16436, R, 256128), (164, 768, 18218, R, 256128), (167, 640, 17369, R, 256128),
    (416, 448, 16852, R, 256160), (389, 448, 19826, R, 256160), (404, 480, 18449, R, 256160),
    (481, 368, 16548, R, 256192), (498, 320, 19890, T, 256192), (487, 320, 20609, T, 256192), (503, 384, 20596, T, 256192), (690, 384, 14538, R, 256192),
    (1010, 272, 15124, R, 256256), (674, 272, 18778, R, 256256), (683, 288, 18737, R, 256256), (583, 384, 19532, R, 256256), (927, 384, 13689, R, 256256),
    (1363, 304, 15332, R, 256384), (2029, 304, 10418, R, 256384), (1253, 288, 19457, R, 256384), (1162, 768, 16620, T, 256384), (1159, 768, 16377, T, 256384)]


@pytest.mark.parametrize("t,c_i,c_o,layout,tile", SHAPES)
def test_ragged_rows_of_every_tile(t, c_i, c_o, layout, tile):
    assert sq.lib().sq_probe_linear_tile(t, c_i, c_o, layout) == 1000000 + tile
    g = torch.Generator(device="cuda").manual_seed(t + c_o)
    x, w = (torch.randint(-127, 128, s, generator=g, device="cuda", dtype=torch.int32).to(torch.int8) for s in ((t, c_i), (c_o, c_i)))
    xs, ws, bias = (torch.rand(n, generator=g, device="cuda") * 0.01 + 0.001 for n in (t, c_o, c_o))
    xq, wq = (_tile(x), _tile(w)) if layout == T else (x, w)
    at = lambda a: (a._base if a._base is not None else a).data_ptr()
    v = (x.double() @ w.double().t()).float() * (xs[:, None] * ws)  # (the integer product exact)
    for dtype in (torch.float16, torch.bfloat16):
        res = torch.randn((t, c_o), generator=g, device="cuda").to(dtype)
        for kind in ("plain", "residual", "in place"):
            print(f"ragged tile {tile} {t}x{c_i}->{c_o} layout {layout} {dtype} {kind}", flush=True)
            want = (v if kind == "plain" else (v + bias).clamp_min(0) + res.float()).to(dtype)
            buf = torch.full((t * c_o + 2 * GUARD,), -7.0, dtype=dtype, device="cuda")
            y = buf[GUARD:GUARD + t * c_o].view(t, c_o)
            if kind == "in place":
                y.copy_(res)
            r = None if kind == "plain" else y.data_ptr() if kind == "in place" else res.data_ptr()
            n = sq.lib().sq_workspace_bytes(2, t, c_i, c_o)
            scratch = torch.empty(max(16, n), dtype=torch.uint8, device="cuda")
            status = sq.lib().sq_w8a8_linear(at(xq), xs.data_ptr(), 1, at(wq), ws.data_ptr(), 1, None if kind == "plain" else bias.data_ptr(), r,
                                             0 if kind == "plain" else 1, y.data_ptr(), sq.BF16 if dtype == torch.bfloat16 else sq.F16, t, c_i, c_o, layout,
                                             scratch.data_ptr(), scratch.numel(), torch.cuda.current_stream().cuda_stream)
            assert status == 0 and torch.equal(y.view(torch.int16), want.view(torch.int16))
            assert bool((buf[:GUARD] == -7.0).all()) and bool((buf[GUARD + t * c_o:] == -7.0).all())
