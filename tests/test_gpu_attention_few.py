"""The few-query form of the fused attention (16-row blocks; taken by a time model for few queries, or few heads) against
the oracle's chain, at the edges of its row blocks, 64-key groups and register sizes (4 or 8 waves, 2 / 4 / 8 / 16 groups
each); and shapes around the model's border with the row-block form, with scores that leave the range of a fixed shift.
Gates as for the row-block form: codes within one, at most one in a thousand; the output identical to the oracle's P V of
the kernel's own codes."""
import numpy as np
import pytest
import torch

import oracle
from paper_2211_10438_amd import binding as sq
from tests._util import BF16, F16, assert_identical_16, bits_from_dev, dev, torch_dtype, ulp_distance

pytestmark = pytest.mark.gpu

# (b, s_q, s_k, d); up to 256 workgroups run eight waves, more (or 4097 keys and up never) four
CASES = [(1, 1, 16, 128), (2, 1, 64, 64), (3, 15, 80, 128), (2, 16, 512, 64), (2, 17, 528, 128), (1, 64, 1024, 128), (1, 64, 1040, 64),
         (1, 65, 1040, 64), (2, 2, 2064, 128), (1, 3, 4112, 64), (1, 1, 8192, 128), (1, 1, 8208, 64),
         (260, 1, 80, 128), (257, 1, 272, 64), (300, 2, 528, 128), (70, 50, 512, 64), (260, 1, 2064, 64), (258, 1, 4096, 128),
         (258, 1, 4112, 64),
         # row blocks of 128: many heads per query row, a last block of few rows, a last tile of one 16-key group, key counts
         # on and off the 64- and 128-key tiles
         (60, 129, 144, 128), (60, 137, 272, 64), (50, 190, 192, 128), (33, 300, 320, 128), (40, 200, 208, 64)]


def _codes(shape, seed):
    x = np.random.default_rng(seed).standard_normal(shape, dtype=np.float32)
    return np.clip(np.rint(x * np.float32(127.0 / 4.5)), -127, 127).astype(np.int8)


def _check(q, k, v, alpha1, causal, odt):
    b, s_q, d = q.shape
    s_k = k.shape[1]
    alpha2 = 4.5 / 127.0 / 127.0
    tdt = torch_dtype(odt)
    pq = torch.full((b, s_q, s_k), -128, dtype=torch.int8, device="cuda")
    o = sq.w8a8_attention(dev(q), dev(k), dev(v), alpha1, alpha2, tdt, p_codes=pq, causal=causal)
    o_plain = sq.w8a8_attention(dev(q), dev(k), dev(v), alpha1, alpha2, tdt, causal=causal)
    assert torch.equal(o.view(torch.int16), o_plain.view(torch.int16))
    sc = oracle.w8a8_bmm(q, k, True, alpha1, odt)
    ref = (oracle.softmax_quant_p_causal if causal else oracle.softmax_quant_p)(sc, odt).astype(np.int32)
    got = pq.cpu().numpy().astype(np.int32)
    assert got.min() >= 0, "a code was not written"
    diff = np.abs(got - ref)
    assert diff.max() <= 1 and (diff != 0).mean() <= 1e-3, f"codes: max diff {diff.max()}, rate {(diff != 0).mean():.2e}"
    assert_identical_16(ulp_distance(bits_from_dev(o), oracle.w8a8_bmm(pq.cpu().numpy(), v, False, alpha2, odt)))


@pytest.mark.parametrize("b,s_q,s_k,d", CASES)
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("odt", [F16, BF16])
def test_few_queries_vs_oracle_chain(b, s_q, s_k, d, causal, odt):
    print(f"[case] few queries b={b} s_q={s_q} s_k={s_k} d={d} causal={causal} dtype={odt}", flush=True)
    q, k, v = (_codes((b, n, d), 700 + i + n) for i, n in enumerate((s_q, s_k, s_k)))
    _check(q, k, v, (4.5 / 127.0) ** 2 / d ** 0.5, causal, odt)


@pytest.mark.parametrize("kind", ["first", "last", "equal"])
@pytest.mark.parametrize("odt", [F16, BF16])
def test_few_queries_extreme_rows(kind, odt):
    """One key that holds all the probability (in the first or the last wave's groups: every other lane's sum is rescaled
    to nothing), and scores that are all alike."""
    print(f"[case] few queries extreme rows {kind} dtype={odt}", flush=True)
    b, s_q, s_k, d = 2, 5, 1040, 128
    q, k, v = (_codes((b, n, d), 720 + i) for i, n in enumerate((s_q, s_k, s_k)))
    if kind == "equal":
        _check(q, k, v, 1e-12, True, odt)
        return
    j = 0 if kind == "first" else s_k - s_q  # visible to every row
    q[:] = np.abs(q)
    k[:, j] = 127
    _check(q, k, v, (4.5 / 127.0) ** 2 / d ** 0.5, True, odt)


@pytest.mark.parametrize("b,s_q,s_k,d", [(60, 160, 320, 128), (60, 144, 384, 64)])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("odt", [F16, BF16])
def test_row_blocks_scores_far_above_the_first_tile(b, s_q, s_k, d, causal, odt):
    """The maximum moves by hundreds from tile to tile: every earlier sum is rescaled to nothing."""
    print(f"[case] rising scores b={b} s_q={s_q} s_k={s_k} d={d} causal={causal} dtype={odt}", flush=True)
    q, k, v = (_codes((b, n, d), 740 + i) for i, n in enumerate((s_q, s_k, s_k)))
    q = np.maximum(np.abs(q), 20)
    for j in range(64, s_k, 32):
        k[:, j] = min(127, 30 + j // 4)
    _check(q, k, v, 0.05, causal, odt)


@pytest.mark.parametrize("s_q,s_k,d", [(100, 400, 128), (130, 1040, 128), (256, 256, 64), (48, 528, 64)])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("odt", [torch.float16, torch.bfloat16])
def test_both_forms_give_the_same_codes(s_q, s_k, d, causal, odt):
    """Two heads alone take the few-query form, the same heads among 700 the row-block form; sums and folds run in the same
    order in both, so codes and outputs are the same bit for bit."""
    print(f"[case] both forms s_q={s_q} s_k={s_k} d={d} causal={causal} {odt}", flush=True)
    q, k, v = (dev(_codes((2, n, d), 760 + i)) for i, n in enumerate((s_q, s_k, s_k)))
    few, rows = 2, 700
    out = []
    for b in (few, rows):
        pq = torch.full((b, s_q, s_k), -128, dtype=torch.int8, device="cuda")
        o = sq.w8a8_attention(*(x.repeat(b // 2, 1, 1) for x in (q, k, v)), (4.5 / 127.0) ** 2 / d ** 0.5, 1e-3, odt, p_codes=pq,
                              causal=causal)
        out.append((pq[:2].clone(), pq[-2:].clone(), o[:2].view(torch.int16).clone()))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][0], out[1][1])
    assert torch.equal(out[0][2], out[1][2])
