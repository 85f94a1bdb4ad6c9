"""Row kernels at the edges of their launch rules against fp64: LayerNorm + quantization (one row per wave up to 2048
channels, then 2 to 6 vectors per thread by row count and width) and the cross-lane reductions all of them share.
Gates as in the parity tests: codes within one, at most one in a thousand; steps to 1e-5."""
import pytest
import torch

from paper_2211_10438_amd import binding as sq

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
