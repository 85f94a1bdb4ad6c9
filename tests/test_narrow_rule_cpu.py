"""Which linear layers count as few tokens and few output channels (no GPU work): those ask for no workspace and always run the direct
kernel; the line is part of the interface.  The other sizes here go by the planner's models (test_linear_choice_cpu.py)."""
import pytest

from paper_2211_10438_amd import binding as sq

R, T = sq.ROW_MAJOR, sq.TILED


@pytest.mark.parametrize("t,c_i,c_o,layout,taken", [
    (16, 768, 3072, T, 1),
    (16, 768, 3072, R, 1),
    (32, 768, 3072, R, 0),
    (32, 896, 768, R, 0),
    (48, 1024, 256, R, 0),
    (32, 784, 3072, R, 1),
    (100, 784, 4088, R, 1),
    (100, 768, 4088, R, 0),
    (64, 12288, 4088, T, 1),
    (64, 20480, 4088, T, 0),
    (64, 24576, 4088, T, 0),
    (16, 5120, 5120, T, 1),
    (16, 1024, 5120, T, 1),
    (1, 1024, 5120, T, 0),
    (1, 1024, 6544, T, 0),
    (1, 64, 5120, T, 1),
    (1, 3072, 5120, T, 1),
    (16, 9216, 9216, T, 0),
    (17, 5120, 5120, T, 0),
    (129, 768, 768, T, 0),
])
def test_few_tokens_and_channels(t, c_i, c_o, layout, taken):
    assert sq.lib().sq_probe_narrow_gemm(t, c_i, c_o, layout) == taken
    if taken:
        assert sq.probe_linear_plan(t, c_i, c_o, layout)[0] == 0
