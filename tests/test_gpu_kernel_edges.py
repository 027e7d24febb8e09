"""Kernels at the edges of their tiles, tables and dispatch ranges, against the oracle or a plain fp32 reference."""
import numpy as np
import pytest
import torch

import csd_inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_11462_amd as P
    P.lib()
    return P


@pytest.mark.parametrize("n", [2, 3, 1024, 1025, 2049, 8191, 8192])
@pytest.mark.parametrize("text", ["one_token", "two_tokens", "few", "all_distinct", "bad_ids"])
def test_bigram_fit_tables(P, n, text):
    """The hash tables of the fit: every pair in one slot, every pair in its own, positions at and across a thread's
    share, ids outside the vocabulary (their pairs do not count).  Whole numbers: bit-exact."""
    from oracle import csd_oracle as O
    V = 9000
    r = np.random.RandomState(n)
    s = {"one_token": lambda: np.full(n, 5), "two_tokens": lambda: r.randint(0, 2, n), "few": lambda: r.randint(0, 40, n),
         "all_distinct": lambda: r.permutation(V)[:n], "bad_ids": lambda: r.randint(-3, 30, n)}[text]().astype(np.int32)
    vocab = 25 if text == "bad_ids" else V
    default = I.default_next_table(vocab, 3)
    if text == "bad_ids":
        want, best = default.numpy().copy(), {}
        ok = [(int(a), int(b)) for a, b in zip(s[:-1], s[1:]) if 0 <= a < vocab and 0 <= b < vocab]
        count = {x: ok.count(x) for x in set(ok)}
        for a, b in ok:                                      # in order: among equal counts the pair seen latest stays
            if count[a, b] >= best.get(a, 0):
                best[a], want[a] = count[a, b], b
    else:
        want = O.bigram_fit(s, vocab, default.numpy())
    got = P.bigram_fit(torch.from_numpy(s).cuda(), vocab, default.cuda().clone())
    assert np.array_equal(got.cpu().numpy(), want)
