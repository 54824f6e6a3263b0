"""The time marginals by contracted series on the GPU (the route of rules whose
times lie close, csrc/ile_series.h) against the FP64 oracle, where the route
can go wrong: every instance of the row contraction (1 to 25 modes), windows
partly and wholly outside the table, windows as long as the table, batches that
cross a chunk, plans of several points, a captured call, and both sides of the
choice between the routes.

Bars as in the two rules' own parity tests: 1e-9 of the largest scale over the
rule's times (times 2 + ln n for the band rule's sinc sums), plus 1e-12."""
import numpy as np
import pytest

from paper_2609_37393_amd import synth

from ._helpers import lnL_scale
from .test_gpu_parity import _mode_set

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ile():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2609_37393_amd import ile as m

    m.load()
    return m


def _scale(oracle_mod, pt, th, times):
    big = np.repeat(th, times.size, axis=1)
    big[5] = np.tile(times, th.shape[1])
    S = lnL_scale(oracle_mod, pt, big).reshape(th.shape[1], times.size)
    return np.where(np.isfinite(S), S, 0.0).max(axis=1)


def _check(ile, oracle_mod, pt, th, rule, fine, idx):
    """Samples idx of the batch th under (t_start, h, n), Simpson or (fine > 0) band."""
    import torch

    t0, h, n = rule
    plan = ile.Plan([pt], [th.shape[1]])
    tht = torch.as_tensor(th, device="cuda").contiguous()
    ll = torch.empty(th.shape[1], dtype=torch.float64, device="cuda")
    sub = th[:, idx]
    if fine:
        plan.lnZ_tband(tht, t0, h, n, fine, lnL_out=ll)
        want, grow = oracle_mod.lnL_tband(pt, sub, t0, h, n, fine), 2.0 + np.log(n)
    else:
        plan.lnZ_tmarg(tht, t0, h, n, lnL_out=ll)
        want, grow = oracle_mod.lnL_tmarg(pt, sub, t0, h, n), 1.0
    got = ll.cpu().numpy()[idx]
    plan.close()
    bar = 1e-9 * grow * _scale(oracle_mod, pt, sub, t0 + h * np.arange(n)) + 1e-12
    assert np.array_equal(np.isnan(got), np.isnan(want))
    ok = np.isfinite(want)
    assert np.all(np.abs(got[ok] - want[ok]) <= bar[ok]), (np.abs(got[ok] - want[ok]) / bar[ok]).max()


@pytest.mark.parametrize("K,M,lmax", [(1, 1, None), (2, 2, None), (2, 4, None), (3, 5, None), (3, 9, None),
                                      (5, 12, 8), (4, 16, None), (8, 21, None), (2, 25, 6)])
def test_row_contraction_instances(ile, oracle_mod, K, M, lmax):
    pt = synth.make_point(K, M, 900, 32768.0, 80.0, 50 + M, lm=None if lmax is None else _mode_set(M, lmax))
    th = synth.prior_samples(150, M)
    th[0, 7] = np.nan
    idx = np.arange(150)
    _check(ile, oracle_mod, pt, th, (-0.004, 1.0 / 32768, 259), 0, idx)
    _check(ile, oracle_mod, pt, th, (-0.004, 1.0 / 8192, 33), 5, idx)


@pytest.mark.parametrize("K,M,lmax", [(3, 7, 3), (2, 8, 4), (3, 11, 3), (3, 12, 3), (2, 13, 4), (8, 14, 4), (5, 17, 4),
                                      (1, 18, 4), (3, 19, 4), (3, 20, 6), (3, 23, 6)])
def test_row_contraction_instances_between(ile, oracle_mod, K, M, lmax):
    """Counts of mode pairs between those above, odd and even numbers of modes."""
    test_row_contraction_instances(ile, oracle_mod, K, M, lmax)


# the table covers +-9.2 ms: windows across its start, its end, all of it and
# beyond, wholly outside, a spacing well under the table's, and off its grid
@pytest.mark.parametrize("rule", [(-0.02, 1.0 / 32768, 401), (0.004, 1.0 / 32768, 401), (-0.05, 1.0 / 16384, 1601),
                                  (0.2, 1.0 / 32768, 65), (-0.002, 0.11 / 32768, 129), (-0.003, 2.37 / 32768, 101),
                                  (-0.001, 1.0 / 32768, 3)])
def test_windows_against_the_table(ile, oracle_mod, rule):
    pt = synth.make_point(3, 9, 603, 32768.0, 60.0, 71)
    th = synth.prior_samples(120, 72)
    _check(ile, oracle_mod, pt, th, rule, 0, np.arange(120))
    if rule[2] <= 64 or rule[2] == 65:
        _check(ile, oracle_mod, pt, th, (rule[0], rule[1], min(rule[2], 64)), 3, np.arange(120))


@pytest.mark.parametrize("fine", [0, 4])
def test_batches_across_chunks(ile, oracle_mod, fine):
    """More samples than one chunk of rows holds, and of coefficients: the
    samples about the chunks' ends."""
    pt = synth.make_point(3, 21, 6554, 32768.0, 100.0, 73)
    n = 120_017
    th = synth.prior_samples(n, 74)
    rule = (-0.009, 1.0 / 4096, 64) if fine else (-0.0095, 1.0 / 32768, 611)
    rows = 8 * 63 + 8 if fine else 618
    inner = (112 << 20) // (8 * 3 * ((rows + 15) // 16 * 16)) // 64 * 64
    outer = (112 << 20) // (8 * (3 * 45 + 1 + (64 if fine else 0)) + 12) // 64 * 64
    idx = np.unique(np.clip(np.concatenate([np.arange(b - 2, b + 3) for b in (0, inner, 2 * inner, outer, n - 3)]),
                            0, n - 1))
    _check(ile, oracle_mod, pt, th, rule, fine, idx)


def test_several_points_and_capture(ile, oracle_mod):
    import torch

    pts = synth.batched_points(3, 75, K=3, nt_range=(400, 3000))
    counts = [2000, 700, 1300]
    th = np.concatenate([synth.prior_samples(c, 80 + i) for i, c in enumerate(counts)], axis=1)
    tht = torch.as_tensor(th, device="cuda").contiguous()
    plan = ile.Plan(pts, counts)
    rule = (-0.002, 1.0 / 32768, 131)
    ll = torch.empty(th.shape[1], dtype=torch.float64, device="cuda")
    z, ne = plan.lnZ_tmarg(tht, *rule, lnL_out=ll)
    s = 0
    for p, c in enumerate(counts):
        sub = th[:, s:s + 60]
        bar = 1e-9 * _scale(oracle_mod, pts[p], sub, rule[0] + rule[1] * np.arange(rule[2])) + 1e-12
        want = oracle_mod.lnL_tmarg(pts[p], sub, *rule)
        assert np.all(np.abs(ll[s:s + 60].cpu().numpy() - want) <= bar)
        s += c
    # captured (stream-ordered working memory) and replayed between eager calls
    out = [torch.empty_like(ll), torch.empty_like(z), torch.empty_like(ne)]
    g = torch.cuda.CUDAGraph()
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=st):
        plan.lnZ_tmarg(tht, *rule, lnZ_out=out[1], neff_out=out[2], lnL_out=out[0])
    for _ in range(3):
        for o in out:
            o.zero_()
        plan.lnZ_tmarg(tht, *rule)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out[0], ll) and torch.equal(out[1], z) and torch.equal(out[2], ne)
    plan.close()


def test_routes_agree_where_the_choice_changes(ile, oracle_mod):
    """Rules just inside and just outside the contracted route (rows kept per
    time about the limit) meet the same bar."""
    pt = synth.make_point(3, 9, 6554, 32768.0, 60.0, 76)
    th = synth.prior_samples(200, 77)
    for rows in (8, 40, 110, 116, 119, 122, 200):  # the line lies near 117 for 9 modes and 200 samples
        _check(ile, oracle_mod, pt, th, (-0.004, rows / 32768, 21), 0, np.arange(200))
