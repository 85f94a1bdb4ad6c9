"""Which kernel a linear layer runs (no GPU work), at sizes where the direct kernel and the others are apart on either side: few K steps
and many outputs, rows of the output off 16 bytes, few steps in the streaming kernels, long rows.  us, direct kernel / the others."""
import pytest
import torch

from paper_2211_10438_amd import binding as sq

R, T = sq.ROW_MAJOR, sq.TILED


@pytest.mark.parametrize("t,c_i,c_o,layout,direct", [
    (997, 64, 14912, R, False),     # 55.2 / 12.5
    (2737, 48, 5824, R, False),     # 55.5 / 10.0
    (226, 64, 22848, R, False),     # 23.1 / 8.7
    (3587, 64, 2368, R, False),     # 34.6 / 11.8
    (872, 256, 7840, R, False),     # 20.2 / 10.8
    (490, 64, 749, R, True),        # 4.9 / 10.7
    (187, 64, 10432, R, True),      # 7.1 / 8.3
    (1943, 192, 24, R, True),       # 4.0 / 8.0
    (463, 640, 2501, R, True),      # 9.6 / 18.3
    (210, 448, 9836, T, True),      # 8.4 / 16.5
    (32, 1088, 31936, T, True),     # 11.9 / 20.0
    (19, 640, 17856, T, True),      # 8.3 / 13.0
    (19, 64, 25653, R, True),       # 5.2 / 8.5
    (96, 1600, 8640, R, True),      # 10.4 / 17.3
    (15, 36336, 1360, R, False),    # 38.2 / 25.0
    (37, 8640, 10576, R, False),    # 37.6 / 34.6
    (13, 18112, 1016, R, True),     # 11.0 / 13.4
    (2048, 12288, 36864, T, False),
    (1, 5120, 20480, T, False),
])
def test_the_faster_kernel_is_taken(t, c_i, c_o, layout, direct):
    assert bool(sq.lib().sq_probe_linear_form(t, c_i, c_o, layout)) == direct


# us with the weights in the last-level cache / in memory: the kernel that runs, then the register-streaming one
@pytest.mark.parametrize("t,c_i,c_o,kernel", [
    (82, 1536, 8727, 0),      # 7.7 / 11.1, 10.1 / 12.3: direct tiles of 32 x 32
    (115, 6016, 5768, 0),     # 16.3 / 22.8, 20.8 / 26.4
    (99, 4864, 5872, 0),      # 12.4 / 17.8, 16.4 / 20.8
    (38, 2944, 8935, 0),      # 1.34, 0.97 of the direct kernel's time: weights that fit the L2s together
    (34, 2432, 8320, 0),      # 7.6 / 11.7, 9.5 / 12.1
    (112, 2368, 6895, 0),     # from memory 14.4, 15.6: slabs of two units, rows off the lines
    (63, 10240, 5552, 1),     # from memory 25.0, 29.3
    (60, 8192, 8240, 1),      # from memory 25.3, 27.7: K splits of the ring
    (102, 9344, 9889, None),  # 46.8 / 47.7, 32.9 / 42.4: and not where those are behind
    (119, 3328, 6560, None),  # 18.6 / 19.8, 13.4 / 17.2: nor slabs of two units on whole lines
])
def test_row_major_streaming_leaves_the_faster_kernel(t, c_i, c_o, kernel):
    plan = sq.probe_linear_plan(t, c_i, c_o, R)
    assert tuple(plan[:2]) == (1, 1) if kernel is None else plan[0] == kernel and (kernel == 0 or plan[1] == 0)


def test_the_sizes_that_reach_a_kernel_by_name():
    from tests.test_gpu_planned_paths import CASES
    for t, c_i, c_o, layout, *plan in CASES:
        assert list(sq.probe_linear_plan(t, c_i, c_o, layout)[:3]) == plan, (t, c_i, c_o, layout)


@pytest.mark.parametrize("t,c_i,c_o,layout", [
    (41, 64, 1802509599, T), (38, 128, 1275606840, T), (126, 64, 571716121, T),
    (30, 64, 1791059052, R), (28, 64, 1442480151, R), (36, 16, 1764709523, R),
    (1 << 29, 16, 1, R), (1480621215, 176, 4, R), (2**31 - 1, 16, 1, R), (2**31 - 1, 64, 3, T), (2, 16, 2**31 - 1, R),
])
def test_no_launch_is_cut(t, c_i, c_o, layout):
    """A launch of 2**32 threads or more is cut without an error: its last outputs stay unwritten."""
    form = sq.lib().sq_probe_linear_form(t, c_i, c_o, layout)
    if form:
        mb, nb, nw = form // 100, form // 10 % 10, form % 10
        assert -(-t // (16 * mb)) * -(-c_o // (16 * nb)) * 64 * nw < 2**32
        assert max(t, c_o) + 16 * mb < 2**31  # the launch counts tiles in 32 bits


@pytest.mark.skipif(torch.cuda.is_available(), reason="passes addresses of nothing")
def test_a_named_form_with_too_many_tiles_is_refused():
    L, one = sq.lib(), 4096
    for t, c_i, c_o in ((1 << 29, 16, 1), (2**31 - 1, 16, 1), (16, 16, 2**31 - 1)):
        assert L.sq_probe_linear_blocks(1, 1, 4, one, one, 0, one, one, 0, None, None, 0, one, sq.F16, t, c_i, c_o, R, None) == 4  # SQ_ERR_UNSUPPORTED
