"""The binding's native calls against its general code: the same outputs (bytes, types, shapes) for what they take, the same exceptions
for what they leave to it; and that they take the one and leave the other, follow the current stream and can be captured."""
import pytest
import torch

from paper_2211_10438_amd import binding as sq

pytestmark = pytest.mark.gpu


@pytest.fixture
def both(monkeypatch):
    sq.lib()
    assert sq._fast is not None
    fast = sq._fast

    class Watched:  # the native calls, counting how often one takes its arguments
        taken = 0

        def __getattr__(self, name):
            def call(*args):
                r = getattr(fast, name)(*args)
                self.taken += r is not None
                return r
            return call

    def run(f, native_takes=True):
        out = []
        watched = Watched()
        for native in (watched, None):
            monkeypatch.setattr(sq, "_fast", native)
            try:
                r = f()
                out.append(tuple(r) if isinstance(r, tuple) else (r,))
            except Exception as e:  # noqa: BLE001 (the kinds are compared)
                out.append((type(e), str(e)))
        monkeypatch.setattr(sq, "_fast", fast)
        if native_takes is not None:
            assert watched.taken == (1 if native_takes else 0)
        torch.cuda.synchronize()
        for a, b in zip(*out):
            if isinstance(a, torch.Tensor):
                assert a.dtype == b.dtype and a.shape == b.shape and a.stride() == b.stride() and (a._base is None) == (b._base is None)
                assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
            else:
                assert a == b
        run.taken = watched.taken
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
    taken = []
    for n, f in enumerate((lambda: sq.quantize_act(x[:, :64], 0), lambda: sq.quantize_act(x, 0, c_i=64), lambda: sq.quantize_act(x, True),  # taken there
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
              lambda: sq.softmax_quant_p(x[:, :20].contiguous()), lambda: sq.ln_quantize(x, one.half(), one), lambda: sq.ln_quantize(x, one, one.cpu()))):
        both(f, native_takes=None)
        taken += [n] * both.taken
    print(taken, flush=True)
    assert taken == [21]  # (a product by NaN is an ordinary call)


def test_native_calls_of_layer_preparation(both):
    """Statistics, smoothing factors and weight codes: taken natively with the general code's results, else left to it."""
    c_i, c_o = 192, 160
    for dt in (torch.float16, torch.bfloat16):
        x, w = torch.randn((40, c_i), device="cuda").to(dt), torch.randn((c_i, c_o), device="cuda").to(dt)
        xm, = both(lambda: sq.act_absmax_per_channel(x))
        wm, = both(lambda: sq.weight_absmax_per_in_channel(w))
        xm, wm = xm.cpu(), wm.cpu()
        xm[3], wm[5] = 0.0, float("nan")
        for alpha in (0.5, 0.8):
            f, _ = both(lambda: sq.smooth_scales(xm, wm, alpha))
        both(lambda: sq.smooth_scales(xm.view(2, -1), wm.view(2, -1), 0.5))
        f = torch.rand(c_i) + 0.5
        for layout in (sq.ROW_MAJOR, sq.TILED):
            for per_channel in (False, True):
                for s in (None, f.cuda()):
                    both(lambda: sq.prepare_weight(w, s, layout=layout, per_channel=per_channel))
    for g in (lambda: sq.act_absmax_per_channel(x[0]), lambda: sq.act_absmax_per_channel(x.t()), lambda: sq.weight_absmax_per_in_channel(w.float()),
              lambda: sq.smooth_scales(xm.cuda(), wm, 0.5), lambda: sq.smooth_scales(xm.double(), wm, 0.5), lambda: sq.smooth_scales(xm[::2], wm[::2], 0.5),
              lambda: sq.smooth_scales(xm, wm, 1), lambda: sq.smooth_scales(xm, wm, 1.5), lambda: sq.smooth_scales(xm[:0], wm[:0], 0.5),
              lambda: sq.prepare_weight(w.float()), lambda: sq.prepare_weight(w, f), lambda: sq.prepare_weight(w.t()), lambda: sq.prepare_weight(w, per_channel=1),
              lambda: sq.prepare_weight(w[:100].contiguous(), layout=sq.TILED), lambda: sq.prepare_weight(w, workspace=torch.empty(4096, dtype=torch.uint8, device="cuda"))):
        both(g, native_takes=False)


def _queue_of_work(stream):
    """A tensor written on `stream` only after some milliseconds of products: what reads it on another stream comes too early."""
    a = torch.randn((8192, 8192), device="cuda").bfloat16()
    b = torch.empty_like(a)
    x = torch.zeros((32, 128), device="cuda").half()
    final = torch.randn((32, 128), device="cuda").half()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for _ in range(30):
            torch.matmul(a, a, out=b)
        x.copy_(final)
    return x, final, (a, b)


def test_native_calls_follow_the_current_stream():
    sq.lib()
    w, one = torch.ones((64, 128), device="cuda", dtype=torch.int8), torch.ones(1, device="cuda")
    gamma = torch.ones(128, device="cuda")
    stream = torch.cuda.Stream()
    x, final, kept = _queue_of_work(stream)
    with torch.cuda.stream(stream):
        xq, xs = sq._fast.quantize_act(x, sq.PER_TOKEN_DYNAMIC, None, None, sq.ROW_MAJOR)
        y = sq._fast.w8a8_linear(xq, xs, w, one, None, None, False, sq.ROW_MAJOR, torch.float16)
        q8 = sq._fast.w8a8_linear_q8(xq, xs, w, one, None, None, False, sq.ROW_MAJOR, torch.float16, one, sq.ROW_MAJOR)
        ln, ls = sq._fast.ln_quantize(x, gamma, gamma, 1e-5, sq.ROW_MAJOR)
        heads = xq.view(2, 16, 128)
        scores = sq._fast.w8a8_bmm(heads, heads, True, 1e-4, torch.float16)
        probs = sq._fast.softmax_quant_p(scores)
        att = sq._fast.w8a8_attention(heads, heads, heads, 1e-4, 1e-3, torch.float16, False)
    busy = not stream.query()  # the calls only queue their work
    torch.cuda.synchronize()
    assert busy
    xq2, xs2 = sq.quantize_act(final, sq.PER_TOKEN_DYNAMIC)
    heads = xq2.view(2, 16, 128)
    scores2 = sq.w8a8_bmm(heads, heads, True, 1e-4, torch.float16)
    want = (xq2, xs2, sq.w8a8_linear(xq2, xs2, w, one, torch.float16), sq.w8a8_linear_q8(xq2, xs2, w, one, one, torch.float16),
            *sq.ln_quantize(final, gamma, gamma), scores2, sq.softmax_quant_p(scores2), sq.w8a8_attention(heads, heads, heads, 1e-4, 1e-3, torch.float16))
    for a, b in zip((xq, xs, y, q8, ln, ls, scores, probs, att), want):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    del kept


def test_native_calls_under_capture():
    """Outputs and workspaces come from the graph's pool; replays on changing inputs, eager work between them."""
    sq.lib()
    t, c_i, c_o = 152, 12736, 2208  # a K split: with a workspace
    assert sq.probe_linear_plan(t, c_i, c_o, sq.TILED)[2] > 1
    w, one = sq.empty_codes(c_o, c_i, sq.TILED), torch.full((1,), 1e-3, device="cuda")
    w.random_(-127, 128)
    x = torch.randn((t, c_i), device="cuda").half()

    def step():
        xq, xs = sq._fast.quantize_act(x, sq.PER_TENSOR_DYNAMIC, None, None, sq.TILED)
        return sq._fast.w8a8_linear(xq, xs, w, one, None, None, True, sq.TILED, torch.float16)

    step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        y = step()
    for n in range(4):
        x.copy_(torch.randn((t, c_i), device="cuda") * (n + 1))
        graph.replay()
        torch.cuda.synchronize()
        got = y.clone()
        assert torch.equal(got.view(torch.int16), step().view(torch.int16)) and float(got.float().max()) > 0
