"""Row-major operands of the direct kernel's small tiles come as two 64-byte loads per 128-byte line: both have to find the line in the
caches.  Sixteen tokens (each weight read by one workgroup) may not take longer than thirty-two (twice the workgroups, the same weights)."""
import pytest
import torch

from paper_2211_10438_amd import binding as sq

pytestmark = pytest.mark.gpu


def _graph(t, c_i, c_o, form):
    g = torch.Generator(device="cuda").manual_seed(t)
    x, w = (torch.randint(-127, 128, s, generator=g, device="cuda", dtype=torch.int32).to(torch.int8) for s in ((t, c_i), (c_o, c_i)))
    xs, ws, y = torch.rand(t, device="cuda"), torch.ones(1, device="cuda"), torch.empty((t, c_o), dtype=torch.float16, device="cuda")

    def call():
        assert sq.lib().sq_probe_linear_blocks(*form, x.data_ptr(), xs.data_ptr(), 1, w.data_ptr(), ws.data_ptr(), 0, None, None, 0, y.data_ptr(), sq.F16,
                                               t, c_i, c_o, sq.ROW_MAJOR, torch.cuda.current_stream().cuda_stream) == 0

    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(10):
            call()
    return graph, (x, w, xs, ws, y)


@pytest.mark.parametrize("c_i,c_o", [(8320, 888), (18112, 1016), (5120, 1664)])
def test_a_line_crosses_once(c_i, c_o):
    # us of 16 / 32 tokens, weights in the caches: 10.7 / 6.3, 19.9 / 8.7 and 8.8 / 5.3 where the first load gave the line up, now 6.2 / 6.3, 8.9 / 9.0
    # and 5.3 / 5.3.  The bound leaves 0.8 us or more for the clock on either side.
    print(f"lines {c_i} -> {c_o}", flush=True)
    graphs = [_graph(t, c_i, c_o, (1, 1, 4)) for t in (16, 32)]
    times = [[], []]
    for n in range(30):
        for (graph, _), out in zip(graphs, times):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            graph.replay()
            b.record()
            torch.cuda.synchronize()
            if n >= 10:
                out.append(a.elapsed_time(b) * 100)
    few, many = (sorted(t)[len(t) // 2] for t in times)
    print(f"{few:.2f} {many:.2f} us", flush=True)
    assert few < 1.15 * many
