"""Each kernel, variant and K split of the linear layer at a size that the planner sends to it, asserted: the tiles in both MFMA shapes and
with K in pairs of steps, their K splits (an odd number of steps each, a short last one, both reduction kernels), the streaming kernels
with and without a K split.  16-bit, int32 and int8 output (rows and tiled) against the exact integer product and the fixed fp32
epilogue in torch: identical."""
import pytest
import torch

from paper_2211_10438_amd import binding as sq
from tests._util import tiled_index
from tests.test_gpu_narrow import _tile

pytestmark = pytest.mark.gpu
R, T = sq.ROW_MAJOR, sq.TILED
STREAM, TILES = 1, 2


def check(t, c_i, c_o, layout, dtype):
    g = torch.Generator(device="cuda").manual_seed(t + c_i + c_o)
    x, w = (torch.randint(-127, 128, s, generator=g, device="cuda", dtype=torch.int32).to(torch.int8) for s in ((t, c_i), (c_o, c_i)))
    xs = torch.rand(t, generator=g, device="cuda") * 0.01 + 0.001
    ws, wsc = torch.full((1,), 3e-4, device="cuda"), torch.rand(c_o, generator=g, device="cuda") * 0.001 + 1e-4
    bias, res = torch.randn(c_o, generator=g, device="cuda"), torch.randn((t, c_o), generator=g, device="cuda").to(dtype)
    acc = (x.double() @ w.double().t()).to(torch.int32)
    xq, wq = (x, w) if layout == R else (_tile(x), _tile(w))
    print("int32", flush=True)
    assert torch.equal(sq.i8_gemm_i32(xq, wq, layout=layout), acc)
    print("plain", flush=True)
    y = sq.w8a8_linear(xq, xs, wq, ws, dtype, layout=layout)
    assert torch.equal(y.view(torch.int16), (acc.float() * (xs[:, None] * ws)).to(dtype).view(torch.int16))
    print("per channel, bias, ReLU, residual", flush=True)
    v16 = ((acc.float() * (xs[:, None] * wsc) + bias).clamp_min(0) + res.float()).to(dtype)
    y = sq.w8a8_linear(xq, xs, wq, wsc, dtype, bias=bias, residual=res, relu=True, layout=layout)
    assert torch.equal(y.view(torch.int16), v16.view(torch.int16))
    if c_o % 8:
        return
    step = torch.full((1,), 0.037, device="cuda")
    r = (torch.ones(1) / torch.full((1,), 0.037)).cuda()  # one IEEE division
    codes = (v16.float() * r).round().clamp(-127, 127).to(torch.int8)
    for out_layout in (R, T) if c_o % 64 == 0 else (R,):
        print("int8", out_layout, flush=True)
        q = sq.w8a8_linear_q8(xq, xs, wq, wsc, step, dtype, bias=bias, residual=res, relu=True, layout=layout, out_layout=out_layout)
        if out_layout == T:
            q = (q._base if q._base is not None else q).reshape(-1)[torch.from_numpy(tiled_index(t, c_o)).cuda()]
        assert torch.equal(q, codes)


# (tokens, C_i, C_o, layout, kernel, variant, K splits)
CASES = [
    # 256 x 256 (0: 32x32x32, 10: 16x16x64), 256 x 192 (6, 12) and 256 x 384 (9, 11); K tails, odd and even steps, long and short K
    (282, 320, 31824, R, TILES, 0, 1), (631, 272, 17392, R, TILES, 0, 1), (266, 320, 30720, T, TILES, 0, 1),
    (278, 1664, 29368, R, TILES, 10, 1), (265, 3328, 29952, T, TILES, 10, 1),
    (410, 304, 16544, R, TILES, 6, 1), (590, 320, 12880, R, TILES, 6, 1), (328, 320, 20864, T, TILES, 6, 1), (406, 11776, 5440, T, TILES, 6, 4),
    (441, 896, 45432, R, TILES, 12, 1), (385, 10496, 22488, R, TILES, 12, 1), (292, 384, 41152, T, TILES, 12, 1), (858, 9984, 11536, T, TILES, 12, 1),
    (266, 304, 44968, R, TILES, 9, 1), (274, 320, 47640, R, TILES, 9, 1), (395, 1088, 41024, T, TILES, 9, 1),
    (417, 1152, 46728, R, TILES, 11, 1), (387, 768, 41408, T, TILES, 11, 1),
    # K splits of the tiles of pairs of steps (13: 256 x 160, 14: 256 x 128, 15: 192 x 224, 16: 192 x 160)
    (583, 6208, 3600, R, TILES, 13, 3), (201, 8576, 1712, R, TILES, 14, 8), (267, 7360, 7088, R, TILES, 15, 3), (151, 11904, 2360, R, TILES, 16, 7),
    (598, 6144, 3717, R, TILES, 13, 3), (212, 13312, 1641, R, TILES, 16, 8), (150, 12160, 2497, R, TILES, 14, 8),
    (409, 6848, 5712, T, TILES, 13, 3), (151, 13696, 2056, T, TILES, 14, 8), (264, 8128, 6912, T, TILES, 15, 3), (135, 9344, 5528, T, TILES, 16, 6),
    (131, 20224, 1728, T, TILES, 14, 8), (140, 9408, 5760, T, TILES, 16, 6), (512, 20480, 5120, T, TILES, 13, 4), (137, 16192, 4237, T, TILES, 16, 8),
    # and of those for few tokens, few and many outputs (one and four columns per thread of the reduction)
    (79, 20928, 1696, R, TILES, 1, 30), (63, 22784, 2152, R, TILES, 2, 30), (4, 15808, 8, R, TILES, 3, 28), (46, 13952, 16, R, TILES, 2, 25),
    (124, 21760, 1072, T, TILES, 1, 31), (64, 26816, 2152, T, TILES, 2, 30), (2, 28096, 8, T, TILES, 3, 32), (66, 12544, 8, T, TILES, 1, 22),
    # streaming, LDS ring (0) and straight into registers (1)
    (1, 512, 16432, R, STREAM, 0, 1), (17, 1024, 16752, R, STREAM, 0, 1), (37, 640, 17720, R, STREAM, 0, 1), (1, 512, 16576, T, STREAM, 0, 1),
    (49, 6080, 4208, R, STREAM, 0, 5), (54, 6656, 4536, R, STREAM, 0, 8), (5, 768, 16512, R, STREAM, 0, 1),
    (33, 1088, 5604, T, STREAM, 1, 1), (53, 1024, 4100, T, STREAM, 1, 1), (104, 1088, 32816, T, STREAM, 1, 1), (64, 8320, 4160, T, STREAM, 1, 5),
    (35, 7296, 8493, T, STREAM, 1, 3), (49, 6912, 4312, T, STREAM, 1, 6), (101, 7488, 8209, T, STREAM, 1, 3),
]


@pytest.mark.parametrize("n", range(len(CASES)))
def test_planned_path(n):
    t, c_i, c_o, layout, kernel, variant, splits = CASES[n]
    assert sq.probe_linear_plan(t, c_i, c_o, layout)[:3] == (kernel, variant, splits)
    print(f"planned path {CASES[n]}", flush=True)
    check(t, c_i, c_o, layout, (torch.float16, torch.bfloat16)[n % 2])
