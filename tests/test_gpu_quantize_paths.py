"""Per-tensor quantization and the calibration statistic at the edges of their launch rules, against the same fixed fp32
arithmetic in torch (every operation of it is exactly rounded, so codes and steps must be identical)."""
import pytest
import torch

from paper_2211_10438_amd import binding as sq
from tests._util import tiled_index

pytestmark = pytest.mark.gpu


def _div(a, b):
    """One IEEE fp32 division on the host (torch turns a division by or of a Python number into a multiplication)."""
    one = lambda v: torch.as_tensor(v, dtype=torch.float32).cpu().reshape(1)  # noqa: E731
    return (one(a) / one(b)).cuda()


def _codes(x, inv_s, r):
    v = x.float() if inv_s is None else x.float() * inv_s
    return (v * r).round().clamp(-127, 127).to(torch.int8)


# rows of 2 and 6 vectors and of two more and two less than 512 and 1024 (the row of a vector comes from a division); 2^21 vectors,
# where two per thread begin, and one row less; a single row, and a tensor of many short rows
@pytest.mark.parametrize("t,c_i", [(1, 16), (3, 48), (70001, 48), (37, 4080), (37, 4112), (513, 8176), (513, 8208), (4095, 4096), (4096, 4096),
                                   (513, 4096), (2049, 8192)])
@pytest.mark.parametrize("with_s", [False, True])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_per_tensor_edges(t, c_i, with_s, dtype):
    print(f"per-tensor {t}x{c_i} s={with_s} {dtype}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(t + c_i)
    full = torch.randn((t, c_i + 8), generator=g, device="cuda").to(dtype)
    x = full[:, :c_i]  # a row stride wider than the row
    full[:, c_i:] = 1e4  # ... whose other columns must not be seen
    full[t - 1, c_i - 1] = 9.0  # the maximum is the tensor's last element
    inv_s = torch.rand(c_i, generator=g, device="cuda") + 0.5 if with_s else None
    v = x.float() if inv_s is None else x.float() * inv_s
    a = v.abs().max()
    small = torch.empty(16, dtype=torch.uint8, device="cuda")
    for ws in (None, small):
        q, step = sq.quantize_act(x, sq.PER_TENSOR_DYNAMIC, inv_s=inv_s, workspace=ws)
        assert torch.equal(step, _div(a, 127.0))
        assert torch.equal(q, _codes(x, inv_s, _div(127.0, a)))
    delta = torch.full((1,), 0.0123, device="cuda")
    q, _ = sq.quantize_act(x, sq.PER_TENSOR_STATIC, inv_s=inv_s, static_scale=delta)
    assert torch.equal(q, _codes(x, inv_s, _div(1.0, delta)))


# few rows take one vector per thread (up to 256 rows, 2064 to 8192 channels), more rows longer threads
@pytest.mark.parametrize("t,c_i", [(1, 2064), (256, 2080), (257, 2080), (2, 8192), (256, 8192), (257, 8192), (3, 8208), (5, 2048)])
@pytest.mark.parametrize("with_s", [False, True])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_per_token_edges(t, c_i, with_s, dtype):
    print(f"per-token {t}x{c_i} s={with_s} {dtype}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(t + c_i)
    x = torch.randn((t, c_i), generator=g, device="cuda").to(dtype)
    x[t - 1, c_i - 1] = 9.0
    inv_s = torch.rand(c_i, generator=g, device="cuda") + 0.5 if with_s else None
    v = x.float() if inv_s is None else x.float() * inv_s
    a = v.abs().amax(1).cpu()
    q, step = sq.quantize_act(x, sq.PER_TOKEN_DYNAMIC, inv_s=inv_s)
    assert torch.equal(step.cpu(), a / torch.full_like(a, 127.0))
    assert torch.equal(q, _codes(x, inv_s, (torch.full_like(a, 127.0) / a).cuda()[:, None]))


# one row range and several (2048 rows each at least), channel counts that end inside a 64-channel column
@pytest.mark.parametrize("t", [1, 31, 129, 2048, 2049, 9000])
@pytest.mark.parametrize("c_i", [16, 64, 1040])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_channel_maxima(t, c_i, dtype):
    print(f"channel maxima {t}x{c_i} {dtype}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(t * 3 + c_i)
    x = torch.randn((t, c_i), generator=g, device="cuda").to(dtype)
    x[t - 1, c_i - 1] = -50.0
    x[0, 0] = 51.0
    assert torch.equal(sq.act_absmax_per_channel(x), x.float().abs().amax(0))


# weight tiles of 64 x 128 per wave and 256 x 128 per workgroup, column slabs of 64 rows and more, 512-column workgroups: one
# piece short of, at and past each edge
@pytest.mark.parametrize("c_i,c_o", [(16, 8), (64, 120), (80, 136), (240, 512), (256, 520), (272, 128), (4160, 264), (320, 4104)])
@pytest.mark.parametrize("per_channel", [False, True])
@pytest.mark.parametrize("with_s", [False, True])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_weight_preparation_edges(c_i, c_o, per_channel, with_s, dtype):
    print(f"weights {c_i}x{c_o} per_channel={per_channel} s={with_s} {dtype}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(c_i + c_o)
    w = (torch.randn((c_i, c_o), generator=g, device="cuda") * 0.02).to(dtype)
    w[c_i - 1, c_o - 1] = -0.5  # the tensor's and its column's maximum is the last element
    w[:, c_o // 2] = 0.0        # a column of zeros: step 0, codes 0
    s = torch.rand(c_i, generator=g, device="cuda") + 0.5 if with_s else None
    v = w.float() if s is None else w.float() * s[:, None]
    a = (v.abs().amax(0) if per_channel else v.abs().max().reshape(1)).cpu()
    r = torch.where(a > 0, torch.full_like(a, 127.0) / a, torch.zeros_like(a)).cuda()
    codes = (v * r).round().clamp(-127, 127).to(torch.int8).t().contiguous()
    for layout in [sq.ROW_MAJOR] + ([sq.TILED] if c_i % 64 == 0 else []):
        wq, step = sq.prepare_weight(w, s, layout=layout, per_channel=per_channel)
        assert torch.equal(step.cpu(), a / torch.full_like(a, 127.0))
        if layout == sq.TILED:
            flat = wq._base.reshape(-1) if wq._base is not None else wq.reshape(-1)
            wq = flat[torch.from_numpy(tiled_index(c_o, c_i)).cuda()]
        assert torch.equal(wq, codes)
    assert torch.equal(sq.weight_absmax_per_in_channel(w), w.float().abs().amax(1))


def test_channel_maxima_of_a_row_longer_than_one_grid():
    """2^30 channels and a few: a workgroup per 64 channels would be 2^24 workgroups of 256 threads, more than a launch takes."""
    print("channel maxima of one very long row", flush=True)
    c_i = (1 << 30) + 48
    x = torch.zeros((1, c_i), dtype=torch.float16, device="cuda")
    x[0, ::4099] = -3.0
    x[0, -1] = 5.0
    out = sq.act_absmax_per_channel(x)
    assert float(out[-1]) == 5.0 and torch.equal(out.half(), x[0].abs())


def test_weight_maxima_of_more_rows_than_one_grid():
    """2^26 rows and a few: one per wave would be 2^24 workgroups of 256 threads, more than a launch takes."""
    print("weight maxima of very many rows", flush=True)
    c_i = (1 << 26) + 5
    w = torch.zeros((c_i, 8), dtype=torch.float16, device="cuda")
    w[::4099, 3] = -3.0
    w[-1, 7] = 5.0
    out = sq.weight_absmax_per_in_channel(w)
    assert float(out[-1]) == 5.0 and torch.equal(out.half(), w.abs().amax(1))


# one wave per row, four waves per row (few long rows; another line with the tensor's maximum), rows on both sides of each
@pytest.mark.parametrize("c_i,c_o", [(16, 4096), (16, 4104), (1024, 4104), (1040, 4104), (48, 8200), (256, 16384), (256, 16392), (272, 16392)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_weight_row_maxima_edges(c_i, c_o, dtype):
    print(f"weight row maxima {c_i}x{c_o} {dtype}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(c_i + c_o)
    w = (torch.randn((c_i, c_o), generator=g, device="cuda") * 0.02).to(dtype)
    w[c_i - 1, c_o - 1] = -0.5
    w[0, 0] = 0.4
    s = torch.rand(c_i, generator=g, device="cuda") + 0.5
    assert torch.equal(sq.weight_absmax_per_in_channel(w), w.float().abs().amax(1))
    _, step = sq.prepare_weight(w, s)
    assert torch.equal(step, _div((w.float() * s[:, None]).abs().max(), 127.0))


@pytest.mark.parametrize("offset", [4, 8, 16])
def test_workspace_of_the_stated_size_needs_word_alignment_only(offset):
    """The stated bytes at any word boundary hold one maximum for each workgroup (two launches), and nothing beyond them is written."""
    t, c = 129, 4096
    print(f"per tensor workspace at offset {offset}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(offset)
    x = torch.randn((t, c), generator=g, device="cuda", dtype=torch.float16)
    need = sq.workspace_bytes(sq.OP_QUANTIZE_ACT, t, c, 0)
    room = torch.full((offset + need + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    q, step = sq.quantize_act(x, sq.PER_TENSOR_DYNAMIC, workspace=room[offset:offset + need])
    ref, ref_step = sq.quantize_act(x, sq.PER_TENSOR_DYNAMIC)
    assert torch.equal(q, ref) and torch.equal(step, ref_step) and torch.equal(step, _div(x.abs().max(), 127.0))
    words = (room != 0xA5).view(-1, 4).any(1)
    assert words[offset // 4:][:need // 4].sum() > 8  # (three launches write one word)
    assert not words[:offset // 4].any() and not words[(offset + need) // 4:].any()
