"""Host-side decisions of the fused attention (no GPU work): which row block a workgroup of the causal row-block form takes --
every block of every head once, and the work spread over the 8 XCDs whatever the number of heads is -- and which form is taken."""
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


# (heads, queries, keys, head dimension, causal) where the two forms are far apart, us few queries / row blocks
@pytest.mark.parametrize("b,s_q,s_k,d,causal,form", [
    (768, 1, 2048, 128, 1, 2),    # 66 / 139
    (1, 8192, 8192, 128, 1, 2),   # 111 / 212
    (13, 320, 320, 64, 0, 2),     # 7.7 / 10.4
    (20, 208, 1040, 64, 0, 2),    # 13.4 / 24.9
    (12, 512, 512, 64, 1, 2),     # 8.2 / 14.2
    (51, 208, 208, 128, 0, 1),    # 13.9 / 10.5
    (42, 320, 320, 128, 0, 1),    # 18.9 / 12.9
    (128, 100, 512, 128, 0, 1),   # 24.3 / 16.1
    (123, 208, 1040, 64, 0, 1),   # 34 / 26
    (200, 100, 512, 64, 0, 1),    # 17.4 / 12.4
    (89, 144, 256, 128, 0, 1),    # 17.2 / 9.9
    (82, 320, 320, 64, 0, 1),     # 18.3 / 10.8
    (1, 12, 96, 64, 0, 1),        # 5.5 / 4.8
    (153, 27, 160, 64, 0, 1),     # 7.7 / 6.7
    (6, 100, 128, 128, 1, 2),     # 6.7 / 8.7: the row blocks' diagonal
    (4, 8192, 8192, 128, 1, 1),   # 363 / 219
    (5, 5008, 5008, 128, 1, 1),   # 196 / 134
    (12, 2048, 2048, 128, 1, 1),  # 66 / 58
    (768, 2048, 2048, 128, 1, 1),
    (1, 1, 8208, 128, 0, 1),      # more keys than the few-query form holds
])
def test_the_faster_form_is_taken(b, s_q, s_k, d, causal, form):
    assert sq.lib().sq_probe_attention_form(b, s_q, s_k, d, causal) == form
