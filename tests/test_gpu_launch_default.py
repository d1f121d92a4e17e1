"""The default elements per workgroup of curved Navier-Stokes meshes: one at
N = 4 and on meshes of at most 1,024 elements, two on larger ones at N = 3
(both sides of the line), and the right-hand side at the line is the same for
either (bitwise)."""
import numpy as np
import pytest

from paper_2511_17551_amd import workloads as W
from tests.helpers import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dgx():
    import torch
    assert torch.cuda.is_available()
    from paper_2511_17551_amd import dgx as mod
    return mod


@pytest.mark.parametrize("N,n,epb", [(3, 10, 1), (3, 11, 2), (4, 3, 1), (4, 11, 1)])
def test_curved_ns_default(dgx, N, n, epb):
    c = W.curved_periodic_case(n=n, N=N, eq=W.EQ_NS, mu=2e-3)
    s = dgx.Solver(c)
    u = to_dev(c.u0)
    assert dgx.dgx_get_launch(s.ctx)[0] == epb
    du = to_host(s.rhs(u))
    dgx.dgx_set_launch(s.ctx, 3 - epb, 0)
    assert np.array_equal(to_host(s.rhs(u)), du)
    s.check()
    s.close()
