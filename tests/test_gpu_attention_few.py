"""The two forms of the fused attention, each by name, against the oracle's chain: blocks of 16 queries with the keys dealt to 4
or 8 waves in groups of 128 (2, 4 or 8 groups per wave), and blocks of 128 queries.  (A time model chooses between them, so
that a shape alone does not say which of them a call reaches.)  Gates as for the public entry points: codes within one, at most
one in a thousand; the output identical to the oracle's P V of the kernel's own codes; and both forms, and the one the library
chooses, give the same codes and outputs bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2211_10438_amd import binding as sq
from tests._util import BF16, F16, assert_identical_16, bits_from_dev, dev, torch_dtype, ulp_distance

pytestmark = pytest.mark.gpu

ROWS, FEW = 1, 2

# (b, s_q, s_k, d); up to 256 workgroups and beyond 4096 keys eight waves, else four
CASES = [(1, 1, 16, 128), (2, 1, 64, 64), (3, 15, 80, 128), (2, 16, 512, 64), (2, 17, 528, 128), (1, 64, 1024, 128), (1, 64, 1040, 64),
         (1, 65, 1040, 64), (2, 2, 2064, 128), (1, 3, 4112, 64), (1, 1, 8192, 128),
         (260, 1, 80, 128), (257, 1, 272, 64), (300, 2, 528, 128), (70, 50, 512, 64), (260, 1, 2064, 64), (258, 1, 4096, 128),
         (258, 1, 4112, 64)]

# Row blocks: key counts on and off the 64- and 128-key tiles (one 16-key group in the last, several tiles), a last block of one
# row, of one, two and three 32-row groups (the other waves idle), heads below, at and above the 8 XCDs
ROW_CASES = [(1, 1, 16, 128), (2, 16, 48, 64), (3, 33, 64, 64), (2, 64, 80, 128), (2, 128, 128, 128), (3, 129, 144, 128), (2, 137, 272, 64),
             (1, 190, 192, 128), (2, 300, 320, 128), (2, 200, 208, 64), (8, 96, 256, 64), (9, 100, 256, 128), (1, 257, 640, 64),
             (2, 300, 384, 128), (12, 130, 400, 128), (1, 512, 1024, 64), (1, 777, 1040, 64), (2, 385, 1152, 128), (1, 70, 8208, 128),
             (1, 9, 8320, 64)]


def _codes(shape, seed):
    x = np.random.default_rng(seed).standard_normal(shape, dtype=np.float32)
    return np.clip(np.rint(x * np.float32(127.0 / 4.5)), -127, 127).astype(np.int8)


def _check(form, q, k, v, alpha1, causal, odt):
    b, s_q, d = q.shape
    s_k = k.shape[1]
    alpha2 = 4.5 / 127.0 / 127.0
    tdt = torch_dtype(odt)
    args = (dev(q), dev(k), dev(v), alpha1, alpha2, tdt)
    pq = torch.full((b, s_q, s_k), -128, dtype=torch.int8, device="cuda")
    o = sq.probe_attention(form, *args, p_codes=pq, causal=causal)
    # without the code output, and as the library chooses
    for other in (sq.probe_attention(form, *args, causal=causal), sq.w8a8_attention(*args, causal=causal)):
        assert torch.equal(o.view(torch.int16), other.view(torch.int16))
    sc = oracle.w8a8_bmm(q, k, True, alpha1, odt)
    ref = (oracle.softmax_quant_p_causal if causal else oracle.softmax_quant_p)(sc, odt).astype(np.int32)
    got = pq.cpu().numpy().astype(np.int32)
    assert got.min() >= 0, "a code was not written"
    diff = np.abs(got - ref)
    assert diff.max() <= 1 and (diff != 0).mean() <= 1e-3, f"codes: max diff {diff.max()}, rate {(diff != 0).mean():.2e}"
    assert_identical_16(ulp_distance(bits_from_dev(o), oracle.w8a8_bmm(pq.cpu().numpy(), v, False, alpha2, odt)))


@pytest.mark.parametrize("form,b,s_q,s_k,d", [(FEW, *c) for c in CASES] + [(ROWS, *c) for c in ROW_CASES])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("odt", [F16, BF16])
def test_each_form_vs_oracle_chain(form, b, s_q, s_k, d, causal, odt):
    print(f"[case] form {form} b={b} s_q={s_q} s_k={s_k} d={d} causal={causal} dtype={odt}", flush=True)
    q, k, v = (_codes((b, n, d), 700 + i + n) for i, n in enumerate((s_q, s_k, s_k)))
    _check(form, q, k, v, (4.5 / 127.0) ** 2 / d ** 0.5, causal, odt)


@pytest.mark.parametrize("form", [ROWS, FEW])
@pytest.mark.parametrize("kind", ["first", "last", "equal"])
@pytest.mark.parametrize("odt", [F16, BF16])
def test_extreme_rows(form, kind, odt):
    """One key that holds all the probability (in the first or the last of a row's groups or tiles: every other sum is rescaled
    to nothing), and scores that are all alike."""
    print(f"[case] extreme rows form {form} {kind} dtype={odt}", flush=True)
    b, s_q, s_k, d = 2, 5, 1040, 128
    q, k, v = (_codes((b, n, d), 720 + i) for i, n in enumerate((s_q, s_k, s_k)))
    if kind == "equal":
        _check(form, q, k, v, 1e-12, True, odt)
        return
    j = 0 if kind == "first" else s_k - s_q  # visible to every row
    q[:] = np.abs(q)
    k[:, j] = 127
    _check(form, q, k, v, (4.5 / 127.0) ** 2 / d ** 0.5, True, odt)


@pytest.mark.parametrize("form", [ROWS, FEW])
@pytest.mark.parametrize("b,s_q,s_k,d", [(3, 160, 320, 128), (3, 144, 640, 64)])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("odt", [F16, BF16])
def test_scores_far_above_the_first_tile(form, b, s_q, s_k, d, causal, odt):
    """The maximum moves by hundreds from tile to tile: every earlier sum is rescaled to nothing."""
    print(f"[case] rising scores form {form} b={b} s_q={s_q} s_k={s_k} d={d} causal={causal} dtype={odt}", flush=True)
    q, k, v = (_codes((b, n, d), 740 + i) for i, n in enumerate((s_q, s_k, s_k)))
    q = np.maximum(np.abs(q), 20)
    for j in range(64, s_k, 32):
        k[:, j] = min(127, 30 + j // 4)
    _check(form, q, k, v, 0.05, causal, odt)


@pytest.mark.parametrize("form", [ROWS, FEW])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("odt", [F16, BF16])
def test_largest_sums(form, d, odt):
    """Sums of d products of +-128 (2^21 at d = 128) next to ordinary ones: the row-block form starts its sums at a float's bit
    pattern and reads them as its neighbours."""
    print(f"[case] largest sums form {form} d={d} dtype={odt}", flush=True)
    q, k, v = (_codes((2, n, d), 750 + i) for i, n in enumerate((40, 272, 272)))
    q[:, ::2] = -128
    k[:, 3::7] = -128  # +128 * 128 each with the queries above
    k[:, 5::7] = 127   # -128 * 127
    _check(form, q, k, v, 2.0 ** -19, False, odt)
    _check(form, q, k, v, 2.0 ** -19, True, odt)


@pytest.mark.parametrize("form", [ROWS, FEW])
@pytest.mark.parametrize("alpha1", [2.0 ** 100, 2.0 ** 101, 1.5 * 2.0 ** 101, 3.4e38])
@pytest.mark.parametrize("odt", [torch.float16, torch.bfloat16])
def test_largest_factors(form, alpha1, odt):
    """The row-block form keeps a factor 2^-26 in its scores and clamps alpha1 where it would overflow: a key of score 0 among
    negative ones has all the probability whatever alpha1 is."""
    b, s_q, s_k, d = 1, 3, 272, 64
    q = torch.zeros((b, s_q, d), dtype=torch.int8, device="cuda")
    q[:, :, 0] = 1
    k = torch.zeros((b, s_k, d), dtype=torch.int8, device="cuda")
    k[:, 1:, 0] = -1
    pq = torch.full((b, s_q, s_k), -128, dtype=torch.int8, device="cuda")
    sq.probe_attention(form, q, k, k, alpha1, 1.0, odt, p_codes=pq)
    assert bool((pq[:, :, 0] == 127).all()) and not bool(pq[:, :, 1:].any())


# the last two: several chunks of heads per XCD, with and without heads left over
@pytest.mark.parametrize("b,s_q,s_k,d", [(2, 100, 400, 128), (2, 130, 1040, 128), (9, 256, 256, 64), (3, 48, 528, 64), (272, 1100, 2048, 128),
                                         (277, 1100, 2048, 128)])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("odt", [torch.float16, torch.bfloat16])
def test_both_forms_give_the_same_codes(b, s_q, s_k, d, causal, odt):
    """Sums and folds run in the same order in both, so codes and outputs are the same bit for bit."""
    print(f"[case] both forms b={b} s_q={s_q} s_k={s_k} d={d} causal={causal} {odt}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(760 + s_q)
    q, k, v = ((torch.randn((b, n, d), generator=g, device="cuda") * 28).round().clamp(-127, 127).to(torch.int8) for n in (s_q, s_k, s_k))
    out = []
    for form in (ROWS, FEW):
        pq = torch.full((b, s_q, s_k), -128, dtype=torch.int8, device="cuda")
        o = sq.probe_attention(form, q, k, v, (4.5 / 127.0) ** 2 / d ** 0.5, 1e-3, odt, p_codes=pq, causal=causal)
        out.append((pq, o.view(torch.int16)))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert int(out[0][0].min()) >= 0


def test_forms_are_chosen_by_size_and_refused_where_they_cannot_run():
    form = sq.lib().sq_probe_attention_form
    assert form(768, 1, 2048, 128, 1) == FEW and form(768, 2048, 2048, 128, 1) == ROWS
    assert form(1, 1, 8208, 128, 0) == ROWS  # more keys than the few-query form holds
    q = torch.zeros((1, 1, 64), dtype=torch.int8, device="cuda")
    k = torch.zeros((1, 8208, 64), dtype=torch.int8, device="cuda")
    with pytest.raises(sq.SqmiError, match="unsupported"):
        sq.probe_attention(FEW, q, k, k, 1e-3, 1e-3, torch.float16)
    with pytest.raises(sq.SqmiError, match="unsupported"):
        sq.probe_attention(3, q, k, k, 1e-3, 1e-3, torch.float16)
