"""The row reads of the FP64 data term with the contraction in their shadow,
and the angles' sines, where each can go wrong: mode sets about the groups of
eight and the change of layout, every detector count (padded ones are skipped),
every class of l, windows of four samples, tables past one window of 2^24 rows,
the fixed scratch about its limit, angles beyond the reduction's range.

Bars: FP64 lnL within 1e-9 S + 1e-12 of the oracle, S = |x data| + |x^2 quad|, as
in the parity tests.
The row coordinate u of a table of 2^24 rows has an ulp of 3.7e-9; four roundings
on the way to it move the data term, whose slope is at most pi per row, by
5e-8 S.  Gradients as in their parity tests, 1e-7 (|g| + 1e-6 S + 1e-9), plus the
absolute part of the lnL bar: where the one detector's response vanishes, S and
g fall to 1e-11 and the rounding of the response's own O(1) terms remains."""
import numpy as np
import pytest

from paper_2609_37393_amd import synth

from ._helpers import lnL_scale
from .test_gpu_gradient import oracle_in, to_coords
from .test_gpu_parity import _mode_set

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ile():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2609_37393_amd import ile as m

    m.load()
    return m


def _check(ile, oracle_mod, pt, th, bar=1e-9):
    got = ile.lnL(pt, th).cpu().numpy()
    want = oracle_mod.lnL(pt, th)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    ok = np.isfinite(want)
    S = lnL_scale(oracle_mod, pt, th)
    assert np.all(np.abs(got[ok] - want[ok]) <= bar * S[ok] + 1e-12), np.nanmax(np.abs(got - want)[ok] / S[ok])


@pytest.mark.parametrize("K", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("M,lmax", [(1, None), (7, 3), (8, 3), (9, 3), (12, 4), (13, 4), (13, 8), (16, 4), (17, 4), (21, 4),
                                    (24, 8), (25, 6)])
def test_groups_of_modes_and_detectors(ile, oracle_mod, K, M, lmax):
    pt = synth.make_point(K, M, 500, 32768.0, 60.0, 10 * K + M, lm=None if lmax is None else _mode_set(M, lmax))
    _check(ile, oracle_mod, pt, synth.prior_samples(193, M))


def test_one_sided_modes(ile, oracle_mod):
    """Phases that start above and end below zero."""
    for lm in ([(2, 2), (3, 3)], [(2, -2), (3, -3), (4, -1)], [(4, 4)], [(2, 0), (4, 0)]):
        pt = synth.make_point(2, len(lm), 400, 32768.0, 40.0, 5, lm=np.array(lm))
        _check(ile, oracle_mod, pt, synth.prior_samples(130, 6))


def test_shortest_table(ile, oracle_mod):
    pt = synth.make_point(3, 9, 400, 32768.0, 40.0, 7)
    pt = dict(pt, Q=np.ascontiguousarray(pt["Q"][:, :, 198:202]), t0=pt["t0"] + 198 * pt["dt"])
    th = synth.prior_samples(400, 8)
    th[5] = np.linspace(-8, 8, 400) * pt["dt"]
    _check(ile, oracle_mod, pt, th)


def test_angles_of_any_size(ile, oracle_mod):
    pt = synth.make_point(3, 9, 400, 32768.0, 40.0, 9)
    th = synth.prior_samples(300, 10)
    big = np.array([0.0, -0.0, np.pi / 4, np.pi / 2, -np.pi, 3 * np.pi / 2, 1e-300, 711.0, -1e5, 2.0**30, -(2.0**30) - 1.0,
                    3.3e9, -1e15, 1e300, np.inf])
    for row in (0, 1, 2, 3, 4):
        t = th[:, : big.size].copy()
        t[row] = big
        _check(ile, oracle_mod, pt, t)


def test_table_past_one_window(ile, oracle_mod):
    """Samples on both sides of, and across, row 2^24 of a table."""
    small = synth.make_point(1, 13, 901, 32768.0, 60.0, 11)
    at = 2**24 - 4 - 450  # its middle about the first row of the second window
    Q = np.zeros((1, 13, 2**24 + 2000), np.complex128)
    Q[:, :, at:at + 901] = small["Q"]
    pt = dict(small, Q=Q, t0=small["t0"] - at * small["dt"])
    th = synth.prior_samples(600, 12)
    th[5] = np.linspace(-300, 300, 600) * pt["dt"]
    _check(ile, oracle_mod, pt, th, bar=5e-8)


def test_fixed_scratch_holds_what_it_held(ile, oracle_mod):
    """A 17-mode table of 58 MB as rows of two modes, a third more as the rows of
    eight that are read, is served; one of 72 MB is refused."""
    import ctypes

    import torch

    from .test_zz_no_alloc import ESCRATCH, _call

    lib = ile.load()
    vp, i32, ci = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int
    lib.rift_ile_lnZ_noalloc.argtypes = [ctypes.POINTER(ile.CPoint), i32, vp, vp, vp, vp, vp, vp, ci, vp]
    small = synth.make_point(2, 17, 901, 32768.0, 60.0, 13)
    th = synth.prior_samples(500, 14)
    th[5] = np.linspace(-300, 300, 500) * small["dt"]
    for n_t, fits in ((100_000, True), (125_000, False)):
        Q = np.zeros((2, 17, n_t), np.complex128)
        Q[:, :, n_t - 901:] = small["Q"]
        pt = dict(small, Q=Q, t0=small["t0"] - (n_t - 901) * small["dt"])
        dp = ile.DevicePoint.from_dict(pt)
        t = torch.as_tensor(th, device="cuda").contiguous()
        rc, z, ne, ll = _call(ile, lib.rift_ile_lnZ_noalloc, [dp], [500], t, None, "fp64")
        if fits:
            assert rc == 0
            rc, z1, ne1, l1 = _call(ile, lib.rift_ile_lnZ, [dp], [500], t, None, "fp64")
            assert rc == 0 and np.array_equal(ll, l1)
        else:
            assert rc == ESCRATCH



@pytest.mark.parametrize("K,M,lmax", [(1, 1, None), (2, 5, None), (3, 17, 4), (5, 21, None), (8, 9, None), (6, 25, 8)])
def test_gradient_groups(ile, oracle_mod, K, M, lmax):
    pt = synth.make_point(K, M, 600, 32768.0, 60.0, 40 + K, lm=None if lmax is None else _mode_set(M, lmax))
    th = synth.prior_samples(101, 41)
    th[3] = np.clip(th[3], 0.05, np.pi - 0.05)
    l, g = ile.grad(pt, to_coords(th, 0), coords=0)
    l_or, g_or = oracle_in(oracle_mod, pt, th, 0)
    S = lnL_scale(oracle_mod, pt, th)
    assert np.all(np.abs(l.cpu().numpy() - l_or) <= 1e-9 * S + 1e-12)
    assert np.all(np.abs(g.cpu().numpy() - g_or) <= 1e-7 * (np.abs(g_or) + 1e-6 * S + 1e-9) + 1e-12)
