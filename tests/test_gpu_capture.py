"""dgx_ssprk3_step captured into a HIP graph by the caller, on a stream of its
own: every replay (with eager right-hand sides and synchronisations between
them) leaves the bits that direct calls leave on a second context of the same
history.  Navier-Stokes (gradient pass), the curved mixture shock with limiter
and smoothed blending, and the octree mesh as a grid and as a work list.  A
first step on a mesh, which allocates, is refused under capture and goes
through afterwards."""
import numpy as np
import pytest

from paper_2511_17551_amd import workloads as W
from oracle.thermo import Mixture
from tests.helpers import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dgx():
    import torch
    assert torch.cuda.is_available()
    from paper_2511_17551_amd import dgx as mod
    return mod


def case(which):
    if which == "tgv_ns":
        return W.case_c2(n=4)
    if which.startswith("octree"):
        return W.case_amr(base=4, radii=(0.4, 0.25), centre=(0.45, 0.5, 0.55))
    mix = Mixture(W.Species())
    c = W.case_c3(lambda rs, T: mix.rho_e(rs, T), lambda rs, T: mix.rho_cv(rs, T), n=4)
    c.cfg = dict(c.cfg, positivity=True, alpha_smooth=True)
    return c


@pytest.mark.parametrize("which", ["tgv_ns", "shock", "octree", "octree_worklist"])
def test_replays_are_direct_calls(dgx, which):
    import torch
    c = case(which)
    print("case", which, flush=True)
    a, b = dgx.Solver(c), dgx.Solver(c)
    ua, ub = to_dev(c.u0), to_dev(c.u0)
    dt = dgx.dgx_max_dt(a.ctx, ua, 0.01 if which == "shock" else 0.2)
    dgx.dgx_max_dt(b.ctx, ub, 0.2)
    if which == "octree_worklist":
        for s in (a, b):
            dgx.dgx_set_launch(s.ctx, 2, 2)
    a.ssprk3(ua, dt, 1)
    b.ssprk3(ub, dt, 1)
    du = torch.empty_like(ua)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        b.ssprk3(ub, dt, 2)
    assert np.array_equal(to_host(ub), to_host(ua))  # recorded, not run
    for turn in range(4):
        a.ssprk3(ua, dt, 2)
        graph.replay()
        ga, gb = to_host(ua), to_host(ub)
        assert np.array_equal(gb, ga), (which, turn)
        for s, u in ((a, ua), (b, ub)):  # (a mixture's next solve starts here on both)
            dgx.dgx_rhs(s.ctx, u, 0.0, du)
    assert not np.array_equal(ga, c.u0)
    for s in (a, b):
        s.check()
        s.close()


def test_first_step_is_refused_under_capture(dgx):
    import torch
    c = case("tgv_ns")
    s, ref = dgx.Solver(c), dgx.Solver(c)
    u, v = to_dev(c.u0), to_dev(c.u0)
    x = torch.zeros(8, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        x.add_(1.0)
        with pytest.raises(dgx.DgxError) as ei:
            s.ssprk3(u, 1e-3, 1)
    assert dgx.ERRORS[ei.value.code] == "DGX_E_STATE"
    graph.replay()
    s.ssprk3(u, 1e-3, 1)
    ref.ssprk3(v, 1e-3, 1)
    assert np.array_equal(to_host(u), to_host(v)) and np.array_equal(to_host(x), np.ones(8))
    for t in (s, ref):
        t.check()
        t.close()
