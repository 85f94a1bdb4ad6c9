"""Weight preparation at the edges of its maxima's launch rules: one slab of rows, two, many, more than sixteen; up to 256 parts of the
tensor's maximum, more, the most; a workspace that holds the workgroups' maxima
and one that does not; a workspace aligned to its words only.  Steps and codes against the fixed fp32 arithmetic in torch, identical."""
import pytest
import torch

from paper_2211_10438_amd import binding as sq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("c_i,c_o", [(16, 8), (64, 512), (80, 64), (128, 520), (192, 1032), (4096, 1000), (8208, 72), (256, 16392),
                                     (96, 24), (112, 72), (1024, 200), (1040, 328), (1200, 320), (2048, 600)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_steps_and_codes(c_i, c_o, dtype):
    print(f"weight maxima {c_i}x{c_o} {dtype}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(c_i + c_o)
    w = torch.randn((c_i, c_o), generator=g, device="cuda").to(dtype)
    w[:, 3] = 0
    s = torch.rand(c_i, generator=g, device="cuda") + 0.5
    room = torch.empty(c_o + 64, device="cuda", dtype=torch.float32)
    for sc in (None, s):
        ws = w.float() if sc is None else w.float() * sc[:, None]
        for per_channel in (False, True):
            a = ws.abs().amax(0) if per_channel else ws.abs().amax().reshape(1)
            step = (a.cpu() / torch.tensor(127.0)).cuda()
            r = torch.where(a > 0, (torch.tensor(127.0) / a.cpu()).cuda(), torch.zeros_like(a))
            ref = (ws * r).round().clamp(-127, 127).to(torch.int8).t()
            # the whole workspace; one word per column, off 16 bytes; the least a per-tensor step needs
            for buf in (room, room[1:1 + c_o]) + (() if per_channel else (room[:1],)):
                codes, got = sq.prepare_weight(w, sc, workspace=_raw(buf), per_channel=per_channel) if buf is room else _call(w, sc, buf, per_channel)
                assert torch.equal(got, step) and torch.equal(codes, ref)


def test_many_slabs_of_a_narrow_weight():
    """A tall narrow weight has many slabs: their maxima may not cost more than the maximum of the whole tensor does.  us per channel / per
    tensor: 20.6 / 16.5 where one thread read all slabs of its columns, now 13.7 / 16.5."""
    w = torch.randn((12288, 64), device="cuda").half()
    times = []
    for per_channel in (True, False):
        sq.prepare_weight(w, per_channel=per_channel)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            kept = [sq.prepare_weight(w, per_channel=per_channel) for _ in range(10)]
        out = []
        for n in range(30):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            graph.replay()
            b.record()
            torch.cuda.synchronize()
            if n >= 10:
                out.append(a.elapsed_time(b) * 100)
        times.append(sorted(out)[len(out) // 2])
        del kept
    print(times, flush=True)
    assert times[0] < 1.1 * times[1]


def _raw(t):
    return t.view(torch.uint8)


def _call(w, s, buf, per_channel):
    """The C entry point with a workspace of exactly `buf` (the binding asks for its own size)."""
    c_i, c_o = w.shape
    codes = torch.empty((c_o, c_i), device="cuda", dtype=torch.int8)
    step = torch.empty(c_o if per_channel else 1, device="cuda")
    st = sq.lib().sq_prepare_weight(w.data_ptr(), sq._dt(w), None if s is None else s.data_ptr(), c_i, c_o, codes.data_ptr(), sq.ROW_MAJOR, step.data_ptr(),
                                    int(per_channel), buf.data_ptr(), buf.numel() * 4, sq._stream())
    assert st == 0
    return codes, step
