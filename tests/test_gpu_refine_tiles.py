"""rift_ile_pregrid at the edges of its tiles: one and two native samples past
a 16-sample tile and a 128-sample chunk of halves, odd and even lengths (the
middle sample and the middle phase are their own mirrors), one column tile and
one more, factors beyond one block's four phases.  The bar is that of the
parity test: per series 8 n u Lambda max|q|, nodes bit for bit."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,n,r", [(1, 2, 2), (1, 3, 2), (8, 17, 4), (9, 18, 6), (7, 255, 8), (3, 256, 9), (5, 257, 2),
                                   (2, 258, 64), (1, 513, 33), (40, 33, 10)])
def test_refine_tiles(oracle_mod, S, n, r):
    from paper_2609_37393_amd import ile

    rng = np.random.default_rng(S * 7919 + n * 31 + r)
    q = rng.normal(size=(S, n)) + 1j * rng.normal(size=(S, n))
    got = ile.pregrid(q, r).cpu().numpy()
    want = oracle_mod.pregrid(q, r)
    lam = 2.0 / math.pi * math.log(2 * n) + 2.0
    assert np.all(np.abs(got - want) <= 8 * n * 2.0 ** -53 * lam * np.abs(q).max(axis=-1, keepdims=True))
    assert np.array_equal(got[:, ::r], q)


@pytest.mark.parametrize("S,n,r", [(1, 97, 2), (3, 97, 3), (9, 113, 6), (5, 128, 5), (3, 129, 64), (1200, 81, 10),
                                   (300, 64, 64), (3, 96, 64), (5, 40, 7), (4097, 49, 1)])
def test_refine_forms(oracle_mod, S, n, r):
    """Both forms beside the lines between them, with remainders of series and samples."""
    test_refine_tiles(oracle_mod, S, n, r)


@pytest.mark.parametrize("n,r", [(20, 1), (20, 3), (130, 3)])
def test_nodes_of_a_series_with_an_infinity(n, r):
    """Both forms copy native times: what is not finite reaches neither them nor another series."""
    from paper_2609_37393_amd import ile

    q = np.random.default_rng(n + r).normal(size=(6, n)) + 0j
    clean = ile.pregrid(q, r).cpu().numpy()
    q[2, 7] = np.inf
    got = ile.pregrid(q, r).cpu().numpy()
    assert np.array_equal(got[:, ::r], q)
    others = [0, 1, 3, 4, 5]
    assert np.array_equal(got[others], clean[others])
