"""A plan's working memory over streams: marginals that alternate between two
streams with growing and shrinking rules, on streams that are destroyed and
made again, and eager calls while another stream is being captured.  Every
result is bitwise that of a plan of its own on one stream."""
import numpy as np
import pytest

from paper_2609_37393_amd import synth

pytestmark = pytest.mark.gpu

RULES = {
    "psi": lambda p, t, **kw: p.lnZ_pmarg(t, "trapezoid", 33, **kw),
    "cells": lambda p, t, **kw: p.lnZ_pmarg(t, "cells", **kw),
    "joint": lambda p, t, **kw: p.lnZ_erai(t, 12, 6, **kw),
    "time": lambda p, t, **kw: p.lnZ_tmarg(t, -1e-3, 1 / 32768, 65, **kw),
    "band": lambda p, t, **kw: p.lnZ_tband(t, -2e-3, 1 / 4096, 16, 8, **kw),
}


@pytest.fixture(scope="module")
def case():
    import torch

    from paper_2609_37393_amd import ile

    pt = ile.DevicePoint.from_dict(synth.make_point(3, 9, 1500, 32768.0, 60.0, 51))
    th = torch.as_tensor(synth.prior_samples(20_000, 52), device="cuda").contiguous()
    want = {}
    for name, rule in RULES.items():
        plan = ile.Plan([pt], [th.shape[1]])
        ll = torch.empty(th.shape[1], dtype=torch.float64, device="cuda")
        z, ne = rule(plan, th, lnL_out=ll)
        torch.cuda.synchronize()
        want[name] = (z.clone(), ne.clone(), ll)
        plan.close()
    return pt, th, want


def _same(got, want):
    return all((a == b).all().item() for a, b in zip(got, want))


def test_alternating_streams(case):
    import torch

    from paper_2609_37393_amd import ile

    pt, th, want = case
    plan = ile.Plan([pt], [th.shape[1]])
    torch.cuda.synchronize()
    order = ["psi", "joint", "time", "cells", "band", "joint", "psi", "time"] * 3
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs, done = [], None
    for i, name in enumerate(order):
        st = streams[i % 2]
        with torch.cuda.stream(st):
            if done is not None:  # the plan's partial sums are one set: the caller orders its calls
                st.wait_event(done)
            ll = torch.empty(th.shape[1], dtype=torch.float64, device="cuda")
            z, ne = RULES[name](plan, th, lnL_out=ll)
            done = st.record_event()
        outs.append((name, z, ne, ll))
    torch.cuda.synchronize()
    for name, z, ne, ll in outs:
        assert _same((z, ne, ll), want[name]), name
    plan.close()


def test_streams_made_again(case):
    import torch

    from paper_2609_37393_amd import ile

    pt, th, want = case
    plan = ile.Plan([pt], [th.shape[1]])
    for name in ("psi", "joint", "cells", "time", "band", "psi"):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            ll = torch.empty(th.shape[1], dtype=torch.float64, device="cuda")
            z, ne = RULES[name](plan, th, lnL_out=ll)
        st.synchronize()
        assert _same((z, ne, ll), want[name]), name
        del st
    plan.close()


@pytest.mark.parametrize("name", sorted(RULES))
def test_first_call_beside_a_capture(case, name):
    """The working memory is taken while another stream is being captured."""
    import torch

    from paper_2609_37393_amd import ile

    pt, th, want = case
    plan = ile.Plan([pt], [th.shape[1]])
    ll = torch.empty(th.shape[1], dtype=torch.float64, device="cuda")
    z, ne = torch.empty(1, dtype=torch.float64, device="cuda"), torch.empty(1, dtype=torch.float64, device="cuda")
    x = torch.zeros(1000, device="cuda")
    beside = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, capture_error_mode="global"):
        x += 1.0
        with torch.cuda.stream(beside):
            RULES[name](plan, th, lnL_out=ll, lnZ_out=z, neff_out=ne)
        x += 1.0
    for _ in range(3):
        g.replay()
    torch.cuda.synchronize()
    assert _same((z, ne, ll), want[name]) and (x == 6.0).all().item()
    plan.close()


def test_memory_is_given_back(case):
    import torch

    from paper_2609_37393_amd import ile

    pt, th, want = case
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    for _ in range(8):  # 8 plans of some 100 MB each
        plan = ile.Plan([pt], [th.shape[1]])
        RULES["band"](plan, th)
        RULES["time"](plan, th)
        plan.close()
        torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] >= free - (256 << 20)
