"""The binding's native calls against its general code: the same outputs (bytes, types, shapes) for what they take, the same exceptions
for what they leave to it."""
import pytest
import torch

from paper_2211_10438_amd import binding as sq

pytestmark = pytest.mark.gpu


@pytest.fixture
def both(monkeypatch):
    sq.lib()
    assert sq._fast is not None
    fast = sq._fast

    def run(f):
        out = []
        for native in (fast, None):
            monkeypatch.setattr(sq, "_fast", native)
            try:
                r = f()
                out.append(tuple(r) if isinstance(r, tuple) else (r,))
            except Exception as e:  # noqa: BLE001 (the kinds are compared)
                out.append((type(e), str(e)))
        monkeypatch.setattr(sq, "_fast", fast)
        torch.cuda.synchronize()
        for a, b in zip(*out):
            if isinstance(a, torch.Tensor):
                assert a.dtype == b.dtype and a.shape == b.shape and a.stride() == b.stride() and (a._base is None) == (b._base is None)
                assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
            else:
                assert a == b
        return out[0]

    return run


def test_native_and_general_calls_agree(both):
    g = torch.Generator(device="cuda").manual_seed(3)
    t, c, n = 32, 128, 192  # whole 16-row blocks: every byte of the tiled codes is defined
    for dt in (torch.float16, torch.bfloat16):
        x = torch.randn((t, c), generator=g, device="cuda").to(dt)
        inv_s, step = torch.rand(c, generator=g, device="cuda") + 0.5, torch.full((1,), 0.03, device="cuda")
        w, ws = torch.randint(-127, 128, (n, c), generator=g, device="cuda").to(torch.int8), torch.full((1,), 1e-3, device="cuda")
        wsc, bias, res = torch.rand(n, device="cuda") * 1e-3, torch.randn(n, device="cuda"), torch.randn((t, n), device="cuda").to(dt)
        for layout in (sq.ROW_MAJOR, sq.TILED):
            for mode in (sq.PER_TOKEN_DYNAMIC, sq.PER_TENSOR_DYNAMIC, sq.PER_TENSOR_STATIC):
                for s in (None, inv_s):
                    xq, xs = both(lambda: sq.quantize_act(x, mode, inv_s=s, static_scale=step, layout=layout))
                for kw in ({}, {"bias": bias, "relu": True}, {"residual": res, "bias": bias}):
                    for scale in (ws, wsc):
                        both(lambda: sq.w8a8_linear(xq, xs, w, scale, dt, layout=layout, **kw))
                        both(lambda: sq.w8a8_linear_q8(xq, xs, w, scale, step, dt, layout=layout, out_layout=layout, **kw))
            both(lambda: sq.ln_quantize(x, inv_s, inv_s, layout=layout))
        q, k = (torch.randint(-127, 128, (3, 64, 64), generator=g, device="cuda").to(torch.int8) for _ in range(2))
        scores, = both(lambda: sq.w8a8_bmm(q, k, True, 1e-4, dt))
        p, = both(lambda: sq.softmax_quant_p(scores))
        both(lambda: sq.w8a8_bmm(p, k, False, 1e-3, dt))
        for causal in (False, True):
            both(lambda: sq.w8a8_attention(q, k, k, 1e-4, 1e-3, dt, causal=causal))
    # a row count off 16: the view of the padded storage
    x = torch.randn((5, 64), device="cuda").half()
    sq_f = both(lambda: sq.quantize_act(x, 0)[1])
    assert sq.quantize_act(x, 0, layout=sq.TILED)[0].shape == (5, 64) and sq_f[0].shape == (5,)


def test_what_is_left_to_the_general_code(both):
    x, w = torch.randn((8, 128), device="cuda").half(), torch.zeros((64, 128), device="cuda", dtype=torch.int8)
    one, xq = torch.ones(1, device="cuda"), torch.zeros((8, 128), device="cuda", dtype=torch.int8)
    a = torch.zeros((2, 32, 64), device="cuda", dtype=torch.int8)
    for f in (lambda: sq.quantize_act(x[:, :64], 0), lambda: sq.quantize_act(x, 0, c_i=64), lambda: sq.quantize_act(x, True),  # taken there
              lambda: sq.quantize_act(x.float(), 0), lambda: sq.quantize_act(x.cpu(), 0), lambda: sq.quantize_act(x, 2), lambda: sq.quantize_act(x, 7),
              lambda: sq.quantize_act(x[:, :100].contiguous(), 0), lambda: sq.quantize_act(x, 0, layout=5), lambda: sq.quantize_act(x, 0, inv_s=x),
              lambda: sq.quantize_act(x[:, 0], 0), lambda: sq.quantize_act(x[:0], 0), lambda: sq.quantize_act(x, 0, inv_s=one.cpu()),
              lambda: sq.w8a8_linear(xq, one, w, one, torch.float32), lambda: sq.w8a8_linear(xq, one[:0], w, one, torch.float16),
              lambda: sq.w8a8_linear(xq, one, w[:, :64].contiguous(), one, torch.float16), lambda: sq.w8a8_linear(xq, one, w.t(), one, torch.float16),
              lambda: sq.w8a8_linear(xq, one, w, torch.ones(3, device="cuda"), torch.float16), lambda: sq.w8a8_linear(xq, one, w, one, torch.float16, relu=1),
              lambda: sq.w8a8_linear(xq, one, w, one, torch.float16, residual=x.bfloat16()), lambda: sq.w8a8_linear(x, one, w, one, torch.float16),
              lambda: sq.w8a8_bmm(a, a, True, float("nan"), torch.float16)[:0], lambda: sq.w8a8_bmm(a, a[:, :, :32], True, 1.0, torch.float16),
              lambda: sq.w8a8_attention(a, a, a, -1.0, 1.0, torch.float16), lambda: sq.w8a8_attention(a, a[:1], a, 1.0, 1.0, torch.float16),
              lambda: sq.w8a8_attention(a, a, a, 1, 1, torch.float16), lambda: sq.softmax_quant_p(x.float()),
              lambda: sq.softmax_quant_p(x[:, :20].contiguous()), lambda: sq.ln_quantize(x, one.half(), one), lambda: sq.ln_quantize(x, one, one.cpu())):
        both(f)
