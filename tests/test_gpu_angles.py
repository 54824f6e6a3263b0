"""The polarisation and joint-angle rules on the coefficients of the data pass
(csrc/angles.hip), where the route can go wrong: circles of few, odd and
remainder points, batches that run in several pieces, lanes past a wavefront's
end, mode sets of every degree in phiref, points whose model norm does not
depend on polarisation, and captured calls.

Bars as in the two rules' own parity tests: the largest FP64 scale over the
rule's angles times 1e-9 (polarisation; 1e-9 more for the rules that follow the
maxima) or 1e-8 (joint), plus 1e-12.  A batch in pieces runs the same
arithmetic per sample as a short one: equal bits."""
import numpy as np
import pytest

from paper_2609_37393_amd import synth

from .test_gpu_erai import _bar as _bar_joint
from .test_gpu_pmarg import _bar as _bar_psi
from .test_gpu_pmarg import _compare

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ile():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2609_37393_amd import ile as m

    m.load()
    return m


def _run(ile, pt, th, call):
    import torch

    plan = ile.Plan([pt], [th.shape[1]])
    ll = torch.empty(th.shape[1], dtype=torch.float64, device="cuda")
    call(plan, torch.as_tensor(th, device="cuda").contiguous(), ll)
    got = ll.cpu().numpy()
    plan.close()
    return got


@pytest.mark.parametrize("n_points", [1, 2, 3, 5, 6, 8, 9, 10, 16, 22, 257])
def test_circles_of_few_and_odd_points(ile, oracle_mod, n_points):
    pt = synth.make_point(3, 9, 900, 32768.0, 60.0, 31)
    th = synth.prior_samples(131, 32)
    got = _run(ile, pt, th, lambda p, t, ll: p.lnZ_pmarg(t, "trapezoid", n_points, lnL_out=ll))
    _compare(got, oracle_mod.lnL_pmarg(pt, th, "trapezoid", n_points), _bar_psi(oracle_mod, pt, th, n_points, False),
             n_points)


@pytest.mark.parametrize("n_phi,n_psi", [(1, 1), (2, 2), (3, 1), (5, 9), (9, 6), (33, 17)])
@pytest.mark.parametrize("K,lm", [(1, [(2, 2)]), (2, [(2, 1), (2, -1)]), (3, [(2, 2), (2, -2), (3, 3), (2, 0)]),
                                  (5, None), (8, None)])
def test_joint_grids_by_degree(ile, oracle_mod, K, lm, n_phi, n_psi):
    """Mode sets of largest |m| 1 to 4, grids of one, few, odd and even phases and angles."""
    M = 21 if lm is None else len(lm)
    pt = synth.make_point(K, M, 900, 32768.0, 60.0, 33 + K, lm=None if lm is None else np.array(lm))
    th = synth.prior_samples(67, 34)
    got = _run(ile, pt, th, lambda p, t, ll: p.lnZ_erai(t, n_phi, n_psi, lnL_out=ll))
    _compare(got, oracle_mod.lnL_erai(pt, th, n_phi, n_psi), _bar_joint(oracle_mod, pt, th), (K, M, n_phi, n_psi))


@pytest.mark.parametrize("method,n_points", [("trapezoid", 12), ("laplace", 0), ("cells", 0)])
@pytest.mark.parametrize("snr", [0.5, 3000.0])
def test_faint_and_loud_points(ile, oracle_mod, snr, method, n_points):
    """Amplitudes at which the Laplace rule falls back, and at which a cell is many sigma wide."""
    pt = synth.make_point(2, 4, 900, 32768.0, snr, 35)
    th = synth.prior_samples(200, 36)
    th[0, 7] = np.nan
    th[6, 9] = np.inf  # x = 0: q(u) = 0 everywhere
    got = _run(ile, pt, th, lambda p, t, ll: p.lnZ_pmarg(t, method, n_points, lnL_out=ll))
    want = oracle_mod.lnL_pmarg(pt, th, method, n_points)
    assert np.isnan(got[7])
    _compare(got, want, _bar_psi(oracle_mod, pt, th, n_points, method != "trapezoid"), (snr, method))


@pytest.mark.parametrize("rule", ["joint", "trapezoid", "cells"])
def test_batches_in_pieces(ile, rule):
    """More samples than a piece's coefficients hold (96 MB): every sample as in a short batch."""
    import torch

    rows = 69 if rule == "joint" else 5
    piece = (96 << 20) // (8 * rows)
    n = 2 * piece + 777
    pt = synth.make_point(2, 9, 900, 32768.0, 60.0, 37)
    th = synth.prior_samples(n, 38)

    def call(p, t, ll):
        if rule == "joint":
            return p.lnZ_erai(t, 4, 2, lnL_out=ll)
        return p.lnZ_pmarg(t, rule, 4 if rule == "trapezoid" else 0, lnL_out=ll)

    got = _run(ile, pt, th, call)
    for a in (0, piece - 3000, 2 * piece - 3000, n - 3000):
        b = min(a + 6000, n)
        part = _run(ile, pt, np.ascontiguousarray(th[:, a:b]), call)
        assert np.array_equal(got[a:b], part), (rule, a)
    torch.cuda.empty_cache()


@pytest.mark.parametrize("rule", ["joint", "trapezoid", "laplace", "cells"])
def test_captured_calls_replay(ile, rule):
    import torch

    pts = synth.batched_points(2, 39, K=3, nt_range=(400, 1200))
    counts = [900, 333]
    th = np.concatenate([synth.prior_samples(c, 40 + i) for i, c in enumerate(counts)], axis=1)
    tht = torch.as_tensor(th, device="cuda").contiguous()
    plan = ile.Plan(pts, counts)

    def call(**kw):
        if rule == "joint":
            return plan.lnZ_erai(tht, 6, 4, **kw)
        return plan.lnZ_pmarg(tht, rule, 8 if rule == "trapezoid" else 0, **kw)

    ll = torch.empty(th.shape[1], dtype=torch.float64, device="cuda")
    z, ne = call(lnL_out=ll)
    out = [torch.empty_like(ll), torch.empty_like(z), torch.empty_like(ne)]
    g = torch.cuda.CUDAGraph()
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=st):
        call(lnZ_out=out[1], neff_out=out[2], lnL_out=out[0])
    for _ in range(3):
        for o in out:
            o.zero_()
        call()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out[0], ll) and torch.equal(out[1], z) and torch.equal(out[2], ne)
    plan.close()


@pytest.mark.parametrize("method,n_points", [("cells", 0), ("laplace", 0), ("trapezoid", 64)])
@pytest.mark.parametrize("factor", [0.0, 1e-200, 1e-70, 1e-45, 1e-30, 1e-19, 1e-12])
def test_norm_without_polarisation(ile, oracle_mod, factor, method, n_points):
    """V = 0: q(u) = a + Re(c1 e^{iu}), two stationary points in closed form; and a
    V too small to count beside the data term, where the quartic has roots near
    0 and far out.  The peak lies anywhere on the circle, far above the value at
    u = 0 for most samples."""
    pt = synth.make_point(3, 9, 900, 32768.0, 600.0, 43)
    th = synth.prior_samples(1500, 44)
    with_v, without = dict(pt, V=pt["V"] * factor), dict(pt, V=pt["V"] * 0.0)
    got = _run(ile, with_v, th, lambda p, t, ll: p.lnZ_pmarg(t, method, n_points, lnL_out=ll))
    ref = without if factor < 1e-20 else with_v
    _compare(got, oracle_mod.lnL_pmarg(ref, th, method, n_points),
             _bar_psi(oracle_mod, ref, th, n_points, method != "trapezoid"), (factor, method))


@pytest.mark.parametrize("rule", ["joint", "trapezoid", "laplace", "cells"])
def test_binned_batches_in_pieces(ile, rule):
    """A binned batch of two points, in several pieces of records: every sample as in input order."""
    import torch

    rows = 69 if rule == "joint" else 5
    piece = (96 << 20) // (8 * rows)
    pts = synth.batched_points(2, 45, K=3, nt_range=(400, 1200))
    counts = [piece + 501, piece // 2 + 77]
    th = np.concatenate([synth.prior_samples(c, 46 + i) for i, c in enumerate(counts)], axis=1)
    th[1, 5] = np.nan
    t = torch.as_tensor(th, device="cuda").contiguous()
    out = []
    for binned in (0, 1):
        plan = ile.Plan(pts, counts)
        plan.config = {"sort": binned}
        ll = torch.empty(th.shape[1], dtype=torch.float64, device="cuda")
        if rule == "joint":
            z, ne = plan.lnZ_erai(t, 4, 2, lnL_out=ll)
        else:
            z, ne = plan.lnZ_pmarg(t, rule, 4 if rule == "trapezoid" else 0, lnL_out=ll)
        torch.cuda.synchronize()
        out.append((z.cpu().numpy(), ne.cpu().numpy(), ll.cpu().numpy()))
        plan.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b, equal_nan=True)
    assert np.isnan(out[1][2][5]) and np.isnan(out[1][0][0]) and np.isfinite(out[1][0][1])
