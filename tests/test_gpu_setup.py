"""The model-norm coefficients of a plan's set-up, where their split can go
wrong: every class (l <= 2, 3, 4, 8), one mode, mode sets with gaps in m and of
one parity, padded detectors, and mixed classes in one plan.  At a table of
zeros lnL = -x^2 quad, so the bar is the FP64 bar of the norm alone:
|d lnL| <= 1e-9 x^2 quad + 1e-12, against the oracle."""
import numpy as np
import pytest

from paper_2609_37393_amd import synth

from ._helpers import lnL_scale

pytestmark = pytest.mark.gpu

SETS = [[(2, 2)], [(2, 0)], [(2, -2), (2, 2)], [(2, 1), (2, -1), (2, 0)], [(3, 3), (2, -2), (3, -1)],
        [(4, 4), (4, -4), (3, 1)], [(8, 7), (2, 2), (5, -5), (6, 0)], [(8, 8), (8, -8), (7, 3)]]


@pytest.mark.parametrize("K", [1, 3, 4, 7])
def test_norm_coefficients(oracle_mod, K):
    import torch

    from paper_2609_37393_amd import ile

    pts, ths = [], []
    for j, lm in enumerate(SETS):
        pt = synth.make_point(K, len(lm), 64, 32768.0, 40.0, 60 + j, lm=lm)
        pt["Q"] = np.zeros_like(pt["Q"])
        pts.append(pt)
        ths.append(synth.prior_samples(70, j))
    want = np.concatenate([oracle_mod.lnL(p, t) for p, t in zip(pts, ths)])
    alone = np.concatenate([ile.lnL(p, t).cpu().numpy() for p, t in zip(pts, ths)])
    _, _, mixed = ile.lnZ(pts, torch.as_tensor(np.concatenate(ths, axis=1)), n_per_point=[70] * len(pts),
                          want_lnL=True)
    for got in (alone, mixed.cpu().numpy()):
        assert np.all(np.abs(got - want) <= 1e-9 * np.abs(want) + 1e-12)


@pytest.mark.parametrize("lead,precision", [(1, "fp64"), (5, "mixed")])
def test_mixed_classes_of_long_tables(oracle_mod, lead, precision):
    """Tables too long to share an allocation with the coefficients, a first
    point with l <= 4 and one further on with l > 4."""
    import torch

    from paper_2609_37393_amd import ile

    pts = [synth.make_point(3, 4, 1000, 32768.0, 40.0, 80 + j) for j in range(9)]
    pts[lead] = synth.make_point(3, 3, 1000, 32768.0, 40.0, 99, lm=[(8, 8), (2, 2), (6, -3)])
    ths = [synth.prior_samples(200, 90 + j) for j in range(9)]
    want = np.concatenate([oracle_mod.lnL(p, t) for p, t in zip(pts, ths)])
    z, _, got = ile.lnZ(pts, torch.as_tensor(np.concatenate(ths, axis=1)), n_per_point=[200] * 9, precision=precision,
                        want_lnL=True)
    top = want.reshape(9, 200).max(axis=1, keepdims=True)
    lnZ = (top + np.log(np.exp(want.reshape(9, 200) - top).mean(axis=1, keepdims=True)))[:, 0]
    if precision == "fp64":
        S = np.concatenate([lnL_scale(oracle_mod, p, t) for p, t in zip(pts, ths)])
        assert np.all(np.abs(got.cpu().numpy() - want) <= 1e-9 * S + 1e-12)
    assert np.all(np.abs(z.cpu().numpy() - lnZ) <= 1e-3)
