"""Which kernel a linear layer runs (no GPU work), at sizes where the direct kernel and the others are apart on either side: few K steps
and many outputs, rows of the output off 16 bytes, few steps in the streaming kernels, long rows.  us, direct kernel / the others."""
import pytest

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


def test_the_sizes_that_reach_a_kernel_by_name():
    from tests.test_gpu_planned_paths import CASES
    for t, c_i, c_o, layout, *plan in CASES:
        assert list(sq.probe_linear_plan(t, c_i, c_o, layout)[:3]) == plan, (t, c_i, c_o, layout)
