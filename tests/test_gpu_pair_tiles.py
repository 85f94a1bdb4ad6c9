"""The tiles that take K in pairs of steps (256 x 160, 256 x 128, 192 x 224, 192 x 160), in both layouts: ragged tokens and channels, odd
numbers of steps, a last step of one to three chunks, K splits.  Against the exact integer product and the fixed fp32 epilogue: outputs identical."""
import pytest
import torch

from paper_2211_10438_amd import binding as sq
from tests._util import tiled_index
from tests.test_gpu_narrow import _tile, test_narrow_linear as check_linear

pytestmark = pytest.mark.gpu
R, T = sq.ROW_MAJOR, sq.TILED


@pytest.mark.parametrize("t,c_i,c_o,layout,tile", [
    (563, 560, 11250, R, 1192160), (523, 320, 11048, T, 1192160), (563, 960, 11099, T, 1192160), (772, 848, 10287, R, 1192224), (783, 1344, 10265, T, 1192224),
    (247, 848, 12331, R, 1256128), (493, 512, 14185, T, 1256128), (906, 560, 8313, R, 1256160), (578, 832, 12641, T, 1256160),
    (145, 8144, 4189, R, 8192160), (145, 3600, 8369, R, 3256128), (202, 5520, 10881, R, 3256160), (259, 7376, 6869, R, 3192224)])
def test_pair_tiles(t, c_i, c_o, layout, tile):
    assert sq.lib().sq_probe_linear_tile(t, c_i, c_o, layout) == tile
    for n, dtype in enumerate((torch.float16, torch.bfloat16)):
        for kind in (("plain", "all", "i32") if n == 0 else ("all",)):
            print(f"pair tile {t}x{c_i}->{c_o} {dtype} {kind}", flush=True)
            check_linear(t, c_i, c_o, dtype, kind)


@pytest.mark.parametrize("t,c_i,c_o", [(520, 320, 11048), (770, 1344, 10320), (204, 384, 11328), (769, 832, 8320)])
def test_pair_tiles_int8_out(t, c_i, c_o):
    assert sq.lib().sq_probe_linear_tile(t, c_i, c_o, T) % 1000 in (128, 160, 224)
    for dtype in (torch.float16, torch.bfloat16):
        print(f"pair tile int8 {t}x{c_i}->{c_o} {dtype}", flush=True)
        check_linear(t, c_i, c_o, dtype, "per_channel_q8")


@pytest.mark.parametrize("t,c_i,c_o", [(515, 320, 11072), (769, 832, 8320), (770, 1344, 10304), (204, 384, 11328)])
def test_pair_tiles_int8_out_tiled(t, c_i, c_o):
    assert sq.lib().sq_probe_linear_tile(t, c_i, c_o, T) % 1000 in (128, 160, 224)
    g = torch.Generator(device="cuda").manual_seed(t)
    x, w = (torch.randint(-127, 128, s, generator=g, device="cuda", dtype=torch.int32).to(torch.int8) for s in ((t, c_i), (c_o, c_i)))
    xs, ws, step = torch.rand(t, generator=g, device="cuda") * 0.01 + 0.001, torch.full((1,), 3e-4, device="cuda"), torch.full((1,), 0.05, device="cuda")
    xq, wq = _tile(x), _tile(w)
    rows, tiled = (sq.w8a8_linear_q8(xq, xs, wq, ws, step, torch.float16, relu=True, layout=T, out_layout=o) for o in (R, T))
    whole = t // 16 * 16  # (the padding rows of the last block are undefined)
    assert torch.equal(_tile(rows[:whole].contiguous()).reshape(-1), tiled.reshape(-1)[: whole * c_o])
    flat = (tiled._base if tiled._base is not None else tiled).reshape(-1)
    assert torch.equal(flat[torch.from_numpy(tiled_index(t, c_o)).cuda()], rows)


@pytest.mark.parametrize("t,c_i,c_o,layout,tile", [(523, 320, 11048, T, 1192160), (770, 1344, 10320, T, 1192224), (204, 384, 11328, T, 1256128),
                                                   (906, 560, 8316, R, 1256160), (145, 3600, 8372, R, 3256128)])
def test_pair_tiles_sums_end_with_the_output(t, c_i, c_o, layout, tile):
    """Int32 sums of whole 16-byte pieces: ragged tiles write their rows and columns and nothing else."""
    print(f"pair tile sums {t}x{c_i}->{c_o} layout {layout}", flush=True)
    assert sq.lib().sq_probe_linear_tile(t, c_i, c_o, layout) == tile
    g = torch.Generator(device="cuda").manual_seed(t)
    x, w = (torch.randint(-127, 128, s, generator=g, device="cuda", dtype=torch.int32).to(torch.int8) for s in ((t, c_i), (c_o, c_i)))
    want = (x.double() @ w.double().t()).to(torch.int32)  # (exact: below 2^53)
    xq, wq = (_tile(x), _tile(w)) if layout == T else (x, w)
    flat = lambda a: (a._base if a._base is not None else a).data_ptr()
    n, guard = t * c_o, 1 << 16
    acc = torch.full((n + 2 * guard,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    ws = torch.empty(max(16, sq.lib().sq_workspace_bytes(3, t, c_i, c_o)), dtype=torch.uint8, device="cuda")
    status = sq.lib().sq_i8_gemm_i32(flat(xq), flat(wq), acc.data_ptr() + 4 * guard, t, c_i, c_o, layout, ws.data_ptr(), ws.numel(),
                                     torch.cuda.current_stream().cuda_stream)
    assert status == 0 and torch.equal(acc[guard:guard + n].reshape(t, c_o), want)
    assert torch.all(acc[:guard] == 0x5A5A5A5A) and torch.all(acc[guard + n:] == 0x5A5A5A5A)
