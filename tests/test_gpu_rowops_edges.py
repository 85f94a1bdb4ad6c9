"""Row kernels at the edges of their launch rules against fp64: LayerNorm + quantization (one row per wave up to 2048
channels, then one to four strands per thread by row count and width, many rows per workgroup where there are many) and the
cross-lane reductions all of them share.  Gates as in the parity tests: codes within one, at most one in a thousand; steps to 1e-5."""
import numpy as np
import pytest
import torch

from paper_2211_10438_amd import binding as sq
from tests._util import tiled_to_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("t,c", [(1, 16), (5, 1024), (3, 2048), (5, 2064), (3, 5120), (2, 5136), (3, 12288), (2, 12304), (1, 16384),
                                 (2048, 2064), (2050, 4096), (2048, 4112), (2048, 6144), (2048, 6160), (2049, 9216), (2048, 16384)])
@pytest.mark.parametrize("offset", [0.5, 100.0])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_ln_quantize_edges(t, c, offset, dtype):
    """A mean a hundred times the deviation shows statistics that cancel."""
    print(f"ln {t}x{c} offset={offset} {dtype}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(t + c)
    x = (torch.randn((t, c), generator=g, device="cuda") + offset).to(dtype)
    gamma = torch.randn(c, generator=g, device="cuda")
    beta = torch.randn(c, generator=g, device="cuda") * 0.1
    xd = x.double()
    y = (xd - xd.mean(1, keepdim=True)) / (xd.var(1, unbiased=False, keepdim=True) + 1e-5).sqrt() * gamma.double() + beta.double()
    a = y.abs().amax(1, keepdim=True)
    ref = (y * (127.0 / a)).round().clamp(-127, 127)
    q, step = sq.ln_quantize(x, gamma, beta)
    assert torch.allclose(step.double(), (a / 127.0).reshape(-1), rtol=1e-5, atol=0.0)
    diff = (q.double() - ref).abs()
    assert float(diff.max()) <= 1 and float((diff != 0).double().mean()) <= 1e-3


@pytest.mark.parametrize("lane", list(range(0, 64, 5)) + [63])
def test_row_maximum_is_found_in_every_lane(lane):
    """One row per wave of 512 elements, the maximum in the eight of one lane: step and codes of every other lane follow it."""
    x = torch.full((4, 512), 0.25, dtype=torch.float16, device="cuda")
    x[:, lane * 8 + 3] = -8.0
    q, step = sq.quantize_act(x, sq.PER_TOKEN_DYNAMIC)
    assert torch.equal(step.cpu(), torch.full((4,), 8.0) / torch.full((4,), 127.0))
    want = torch.full((4, 512), 4, dtype=torch.int8, device="cuda")  # round(0.25 * 127 / 8)
    want[:, lane * 8 + 3] = -127
    assert torch.equal(q, want)
    s = torch.full((4, 512), float("-inf"), dtype=torch.float16, device="cuda")
    s[:, lane * 8 + 5] = 0.0
    p = sq.softmax_quant_p(s)
    assert int(p[0, lane * 8 + 5]) == 127 and int(p.to(torch.int32).sum()) == 4 * 127


def _strand_sum(v, strands):
    """fp32 sum of the rows of v [t, vectors, 8] in the kernels' fixed order: vector i to strand i % strands, a strand's elements
    one after the other, 64 neighbouring strands in a butterfly, these sums as (0 + 1) + (2 + 3), then + ((4 + 5) + (6 + 7))."""
    t, nvec, _ = v.shape
    rounds = -(-nvec // strands)
    pad = np.zeros((t, rounds * strands, 8), np.float32)
    pad[:, :nvec] = v
    pad = pad.reshape(t, rounds, strands, 8)
    s = np.zeros((t, strands), np.float32)
    for i in range(rounds):
        for e in range(8):
            s += pad[:, i, :, e]
    s = s.reshape(t, strands // 64, 64)
    for o in (32, 16, 8, 4, 2, 1):
        s = s + s[:, :, np.arange(64) ^ o]
    s = s[:, :, 0]
    if strands == 64:
        return s[:, 0]
    total = (s[:, 0] + s[:, 1]) + (s[:, 2] + s[:, 3])
    if strands == 512:
        total = total + ((s[:, 4] + s[:, 5]) + (s[:, 6] + s[:, 7]))
    return total


# both sides of every width at which the launch changes, few rows and many
@pytest.mark.parametrize("t,c", [(5, 1024), (5, 1040), (3, 2048), (5, 2064), (3, 4096), (3, 4112), (3, 5120), (3, 6144), (3, 6160),
                                 (2, 8192), (2, 8208), (3, 9216), (2, 12288), (2, 12304), (1, 16384), (2049, 2080), (3073, 2064),
                                 (2050, 4096), (3080, 4096), (1601, 5120), (2049, 5136), (3073, 4112), (1401, 6160), (2049, 6160),
                                 (3073, 8192), (1025, 9216), (1537, 8208), (769, 12304), (3585, 4112), (3600, 5120), (4609, 6144),
                                 (513, 2080), (513, 4096), (514, 6144), (513, 8192), (300, 12288), (4099, 528), (4097, 1024), (4098, 1040), (4099, 2048)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_ln_quantize_is_one_fixed_fp32_sequence(t, c, dtype):
    """Every sum, product and quotient rounds by itself and in one order, whatever the launch: steps and codes are identical
    to the same sequence in numpy."""
    print(f"ln sequence {t}x{c} {dtype}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(t * 7 + c)
    x = (torch.randn((t, c), generator=g, device="cuda") + 0.3).to(dtype)
    gamma = torch.randn(c, generator=g, device="cuda")
    beta = torch.randn(c, generator=g, device="cuda") * 0.1
    q, step = sq.ln_quantize(x, gamma, beta)
    v = x.float().cpu().numpy().reshape(t, c // 8, 8)
    n, strands = np.float32(c), 64 if c <= 2048 else 256 if c <= 8192 else 512
    mean = (_strand_sum(v, strands) / n)[:, None, None]
    d = v - mean
    var = _strand_sum(d * d, strands) / n
    rstd = (np.float32(1) / np.sqrt(var + np.float32(1e-5)))[:, None, None]
    y = (d * rstd * gamma.cpu().numpy().reshape(c // 8, 8) + beta.cpu().numpy().reshape(c // 8, 8)).reshape(t, c)
    a = np.abs(y).max(axis=1)
    assert y.dtype == np.float32 and np.array_equal(step.cpu().numpy(), a / np.float32(127))
    assert np.array_equal(q.cpu().numpy(), np.rint(y * (np.float32(127) / a)[:, None]).astype(np.int8))


@pytest.mark.parametrize("t,c,tiled", [(1537, 8208, False), (1537, 12288, True), (2047, 9216, True), (2049, 8256, True), (3585, 4112, False),
                                       (3585, 6144, True), (4607, 5120, False), (4609, 5184, True)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_ln_quantize_many_rows_per_workgroup(t, c, tiled, dtype):
    """Rows that share a workgroup, and the workgroups that have one row more than others: each row's codes and step are those of
    a call with a few rows, in an order of magnitude that changes from row to row."""
    print(f"ln many rows {t}x{c} tiled={tiled} {dtype}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(t + c)
    x = torch.randn((t, c), generator=g, device="cuda").to(dtype) * (torch.arange(t, device="cuda") % 13 + 1)[:, None].to(dtype)
    x[t - 1] = 0
    gamma = torch.randn(c, generator=g, device="cuda")
    beta = torch.randn(c, generator=g, device="cuda") * 0.1
    q, step = sq.ln_quantize(x, gamma, beta, layout=sq.TILED if tiled else sq.ROW_MAJOR)
    codes = tiled_to_rows(q)[:t, :c] if tiled else q.cpu().numpy()
    for r in range(0, t, 1024):
        few, few_step = sq.ln_quantize(x[r:r + 1024].contiguous(), gamma, beta)
        assert torch.equal(step[r:r + 1024], few_step) and np.array_equal(codes[r:r + 1024], few.cpu().numpy())


@pytest.mark.parametrize("t,c,ldx,tiled", [(1, 16, 16, False), (1, 8192, 8192, False), (1, 8208, 8224, False), (16, 1024, 1088, True), (17, 1024, 1024, True),
                                           (4, 8192, 8192, False), (15, 2192, 2200, False), (256, 8192, 8192, True), (257, 8208, 8208, False), (512, 8192, 8192, True),
                                           (513, 8208, 8216, False), (2, 8192, 8192, True), (2, 8208, 8208, False), (4, 8208, 8224, False),
                                           (8, 8192, 8192, True), (8, 8208, 8208, False)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("smooth", [False, True])
def test_quantize_per_tensor_dynamic_edges(t, c, ldx, tiled, dtype, smooth):
    """One workgroup for the tensor, one for each 1024 vectors of it, and the first sizes beyond either (smoothed tensors earlier), full and ragged ranges of the
    maxima; the maximum in the very last element."""
    print(f"per tensor {t}x{c} ldx={ldx} tiled={tiled} {dtype} smooth={smooth}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(t + c)
    full = torch.randn((t, ldx), generator=g, device="cuda").to(dtype)
    full[:, c:] = 99.0  # not part of the tensor
    full[t - 1, c - 1] = -17.0
    inv_s = torch.rand(c, generator=g, device="cuda") * 0.5 + 0.5 if smooth else None
    q, step = sq.quantize_act(full[:, :c], sq.PER_TENSOR_DYNAMIC, inv_s=inv_s, layout=sq.TILED if tiled else sq.ROW_MAJOR)
    v = full[:, :c].float().cpu().numpy()
    if smooth:
        v = v * inv_s.cpu().numpy()
    a = np.abs(v).max()
    assert step.item() == a / np.float32(127)
    codes = tiled_to_rows(q)[:t, :c] if tiled else q.cpu().numpy()
    assert np.array_equal(codes, np.rint(v * (np.float32(127) / a)).astype(np.int8))
