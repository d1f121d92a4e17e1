"""dgx_max_dt on a state whose wave speed is not finite somewhere: refused
with DGX_E_NONPHYSICAL, whether one node is bad (a NaN, or a negative pressure:
the sound speed is no number) or a whole element, and wherever it lies: the
first nodes, the last, and one that a workgroup reaches in a later turn (the
meshes hold more nodes than one turn of the grid, 131,072).  The bound of the
sound state is the same before and after."""
import numpy as np
import pytest

from paper_2511_17551_amd import workloads as W
from oracle.thermo import Mixture
from tests.helpers import to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dgx():
    import torch
    assert torch.cuda.is_available()
    from paper_2511_17551_amd import dgx as mod
    return mod


def case(which):
    if which == "vortex_96":
        return W.case_c1(n=96)
    if which == "euler_13cube":
        return W.case_c2(n=13, eq=W.EQ_EULER)
    mix = Mixture(W.Species())
    return W.case_c4(lambda rs, T: mix.rho_e(rs, T), lambda rs, T: mix.rho_cv(rs, T), nr=8, nth=16, hot=True)


def refused(dgx, s, u):
    with pytest.raises(dgx.DgxError) as ei:
        dgx.dgx_max_dt(s.ctx, to_dev(u), 0.5)
    return dgx.ERRORS[ei.value.code] == "DGX_E_NONPHYSICAL"


@pytest.mark.parametrize("which", ["vortex_96", "euler_13cube", "cylinder_8x16"])
def test_bad_nodes_are_refused(dgx, which):
    c = case(which)
    s = dgx.Solver(c)
    E, nn = c.u0.shape[1:]
    ref = dgx.dgx_max_dt(s.ctx, to_dev(c.u0), 0.5)
    later = min(E - 2, 131072 // nn + 3)
    for e, n in ((0, 0), (later, nn // 2), (E - 1, nn - 1)):
        u = c.u0.copy()
        u[0, e, n] = np.nan
        assert refused(dgx, s, u), ("NaN node", e, n)
        u = c.u0.copy()
        u[:, e] = np.nan
        assert refused(dgx, s, u), ("NaN element", e)
        if which != "cylinder_8x16":
            u = c.u0.copy()
            u[-1, e, n] = 0.5 * (u[1:-1, e, n] ** 2).sum() / u[0, e, n] - 0.1
            assert refused(dgx, s, u), ("negative pressure", e, n)
    # (a mixture's solve starts from the node's last temperature: to rounding)
    assert abs(dgx.dgx_max_dt(s.ctx, to_dev(c.u0), 0.5) - ref) <= (1e-13 * ref if which == "cylinder_8x16" else 0.0)
    s.close()
