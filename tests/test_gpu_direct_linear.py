"""The direct kernel (operands from memory into MFMA registers, K dealt to the waves of a workgroup), every instantiation, at the edges
of its tiles, its share of K per wave and its buffers in flight.  Against the exact integer product and the fixed fp32 epilogue in
torch: outputs identical."""
import pytest
import torch

from paper_2211_10438_amd import binding as sq
from tests.test_gpu_narrow import _tile

pytestmark = pytest.mark.gpu

FORMS = [(1, 1, 2), (1, 1, 4), (1, 2, 2), (1, 2, 4), (1, 4, 2), (1, 4, 4), (2, 2, 2), (2, 2, 4), (2, 4, 4), (3, 2, 4), (3, 4, 4), (4, 4, 4),
         (5, 4, 4), (6, 4, 4), (7, 4, 4)]


def _ptr(t):
    return None if t is None else t.data_ptr()


@pytest.mark.parametrize("mb,nb,nw", FORMS)
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_every_form_at_its_edges(mb, nb, nw, dtype):
    g = torch.Generator(device="cuda").manual_seed(mb * 100 + nb * 10 + nw)
    bm, bn = 16 * mb, 16 * nb
    # one K step and parts of one, an odd number of steps, fewer pairs than waves, a pair more or less than each wave's buffers hold
    ks = [16, 64, 80, 128, 192, 128 * nw, 128 * nw + 48, 128 * nw * 2 + 64, 128 * nw * 4 - 16, 128 * nw * 5 + 192]
    sizes = [(1, 1), (bm - 1, bn + 1), (bm, bn), (bm + 1, 2 * bn - 4), (2 * bm + 5, 3 * bn + 2), (3 * bm, 9 * bn)]
    for n, k in enumerate(ks):
        for m, (t, c_o) in enumerate(sizes):
            print(f"direct {mb}x{nb}x{nw} {dtype} {t}x{k}->{c_o}", flush=True)
            full, per_channel = (n + m) % 3 == 0, (n + m) % 2 == 0
            x, w = (torch.randint(-127, 128, s, generator=g, device="cuda", dtype=torch.int32).to(torch.int8) for s in ((t, k), (c_o, k)))
            xs = torch.rand(t, generator=g, device="cuda") * 0.01 + 0.001
            ws = (torch.rand(c_o, generator=g, device="cuda") * 0.001 + 1e-4) if per_channel else torch.full((1,), 3e-4, device="cuda")
            bias = torch.randn(c_o, generator=g, device="cuda") if full else None
            res = torch.randn((t, c_o), generator=g, device="cuda").to(dtype) if full else None
            v = (x.double() @ w.double().t()).float() * (xs[:, None] * ws)
            if full:
                v = (v + bias).clamp_min(0) + res.float()
            ref = v.to(dtype).view(torch.int16)
            for layout in [sq.ROW_MAJOR] + ([sq.TILED] if k % 64 == 0 else []):
                xq, wq = (x, w) if layout == sq.ROW_MAJOR else (_tile(x), _tile(w))
                y = torch.full((t + 1, c_o), 7.0, device="cuda", dtype=dtype)  # a row behind the output that must stay
                st = sq.lib().sq_probe_linear_blocks(mb, nb, nw, _ptr(xq), _ptr(xs), 1, _ptr(wq), _ptr(ws), int(per_channel), _ptr(bias), _ptr(res),
                                                     int(full), _ptr(y), sq.F16 if dtype == torch.float16 else sq.BF16, t, k, c_o, layout, sq._stream())
                assert st == 0
                assert torch.equal(y[:t].view(torch.int16), ref) and bool((y[t] == 7.0).all())


# Sizes the library sends to it, through the public calls: int32 sums, int8 codes with per-channel steps, one step for all tokens
@pytest.mark.parametrize("t,c_i,c_o", [(200, 1216, 1352), (33, 4096, 4096), (700, 1088, 776), (5, 8736, 8352), (130, 2560, 2064)])
def test_public_calls(t, c_i, c_o):
    from tests.test_gpu_narrow import test_narrow_linear
    assert any(sq.lib().sq_probe_linear_form(t, c_i, c_o, layout) for layout in (sq.ROW_MAJOR, sq.TILED))
    for kind in ("plain", "all", "per_channel_q8", "i32"):
        test_narrow_linear(t, c_i, c_o, torch.float16, kind)


def test_a_form_that_is_not_built_is_refused():
    z = torch.zeros((16, 64), device="cuda", dtype=torch.int8)
    f = torch.ones(16, device="cuda")
    y = torch.empty((16, 16), device="cuda", dtype=torch.float16)
    assert sq.lib().sq_probe_linear_blocks(8, 8, 4, _ptr(z), _ptr(f), 1, _ptr(z), _ptr(f), 0, None, None, 0, _ptr(y), 0, 16, 64, 16, 0, sq._stream()) == 4
