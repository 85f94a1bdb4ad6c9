"""Which linear layers run the kernel for few tokens and few output channels (no GPU work): sizes at which it and the tile and
streaming kernels are apart.  us, this kernel / the others."""
import pytest

from paper_2211_10438_amd import binding as sq

R, T = sq.ROW_MAJOR, sq.TILED


@pytest.mark.parametrize("t,c_i,c_o,layout,taken", [
    (16, 768, 3072, T, 1),     # 4.3 / 6.6
    (16, 768, 3072, R, 1),     # 6.3 / 6.6
    (32, 768, 3072, R, 0),     # 7.1 / 6.8: rows of a multiple of 128 bytes
    (32, 896, 768, R, 0),      # 7.4 / 6.9
    (48, 1024, 256, R, 0),     # 8.8 / 8.3
    (32, 784, 3072, R, 1),     # 5.7 / 7.2
    (100, 784, 4088, R, 1),    # 8.1 / 13.7
    (100, 768, 4088, R, 0),    # 10.1 / 9.0
    (64, 12288, 4088, T, 1),   # 21 / 22.6
    (64, 20480, 4088, T, 0),   # 31.5 / 27.6
    (64, 24576, 4088, T, 0),   # 37 / 30
    (16, 5120, 5120, T, 1),    # 11.4 / 13.1
    (16, 1024, 5120, T, 1),    # 4.8 / 5.9
    (1, 1024, 5120, T, 0),     # 6.6 / 5.9
    (1, 1024, 6544, T, 0),     # 6.7 / 6.0
    (1, 64, 5120, T, 1),       # 3.8 / 4.3
    (1, 3072, 5120, T, 1),     # 9.5 / 9.6
    (16, 9216, 9216, T, 0),    # 24 / 22
    (17, 5120, 5120, T, 0),
    (129, 768, 768, T, 0),
])
def test_the_faster_kernel_is_taken(t, c_i, c_o, layout, taken):
    assert sq.lib().sq_probe_narrow_gemm(t, c_i, c_o, layout) == taken
