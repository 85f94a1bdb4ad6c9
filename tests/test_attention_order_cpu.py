"""Which row block a workgroup of the causal row-block attention takes (no GPU work): every block of every head once, and the
work spread over the 8 XCDs whatever the number of heads is."""
import ctypes

import pytest

from paper_2211_10438_amd import binding as sq


def _places(b, s_q, s_k, d):
    """(XCD, head, row block) of every workgroup, in the order of their start."""
    fn, head, out, block = sq.lib().sq_probe_attention_place, ctypes.c_int64(), [], 0
    while (tile := fn(block, b, s_q, s_k, d, ctypes.byref(head))) >= 0:
        out.append((block % 8, head.value, tile))
        block += 1
    return out


# (heads, queries = keys): fewer heads than XCDs, multiples of eight, one more and one less; heads in one chunk and in several
@pytest.mark.parametrize("b", [1, 2, 3, 7, 8, 9, 12, 16, 17, 23, 100])
@pytest.mark.parametrize("s,d", [(100, 64), (128, 128), (384, 128), (1000, 64), (2048, 128), (16384, 128)])
def test_causal_order_is_complete_and_spread_over_the_xcds(b, s, d):
    places, tiles = _places(b, s, s, d), (s + 127) // 128
    assert sorted(p[1:] for p in places) == [(h, t) for h in range(b) for t in range(tiles)]
    work = [0] * 8  # key tiles: row block t sees t + 1
    for xcd, _, tile in places:
        work[xcd] += tile + 1
    # eight ranks of a head dealt to eight XCDs differ by seven key tiles
    assert max(work) - min(work) <= tiles
