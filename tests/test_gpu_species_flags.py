"""Mixture kernels on both forms of the species table: the molecules first
(N2, O2, NO, N, O) and other molecule flags, with temperatures from 200 K to
9000 K between neighbouring nodes, so that every range of the mixture's
means and exponentials occurs (density ratios up to 1e9, theta [[1/T]]/2 on
both sides of 1)."""
import numpy as np
import pytest

from oracle.dgsem import Operator
from oracle.thermo import Mixture
from paper_2511_17551_amd import workloads as W
from tests.helpers import flux_scale, parity_err, to_dev, to_host

pytestmark = pytest.mark.gpu
FLAGS = {"first": ([1, 1, 1, 0, 0], [3393.0, 2273.0, 2739.0, 0.0, 0.0]),
         "mixed": ([1, 0, 1, 0, 1], [3393.0, 0.0, 2739.0, 0.0, 1500.0])}


@pytest.fixture(scope="module")
def dgx():
    import torch
    assert torch.cuda.is_available()
    from paper_2511_17551_amd import dgx as mod
    return mod


def rough_case(flags, vf, sf):
    sp = W.Species(molecule=np.array(FLAGS[flags][0], np.int32), theta_v=np.array(FLAGS[flags][1]))
    mix = Mixture(sp)
    c = W.curved_periodic_mixture_case(lambda rs, T: mix.rho_e(rs, T), n=2, N=4, volume_flux=vf, surface_flux=sf)
    rng = np.random.default_rng(4)
    shape = c.u0.shape[1:]
    T = 10.0 ** rng.uniform(np.log10(200.0), np.log10(9000.0), shape)
    low = np.array([-1.0, -1.0, -9.0, -9.0, -9.0])[:, None, None]
    rs = 0.1 * 10.0 ** (low * rng.uniform(0.0, 1.0, (5,) + shape))
    v = rng.uniform(-300.0, 300.0, (3,) + shape)
    rho = rs.sum(0)
    c.u0 = np.concatenate([rs, rho * v, (mix.rho_e(rs, T) + 0.5 * rho * (v * v).sum(0))[None]])
    c.species = sp
    return c, T


@pytest.mark.parametrize("flags", list(FLAGS))
@pytest.mark.parametrize("vf,sf", [(W.VF_DUCROS, W.SF_RUSANOV), (W.VF_RANOCHA, W.SF_RUSANOV), (W.VF_RANOCHA, W.SF_RANOCHA)])
def test_rough_mixture_rhs(dgx, flags, vf, sf):
    """Right-hand side within 1e-11 of the flux scale (the bound of the flux tests), T(e) within 1e-12."""
    import torch
    c, T = rough_case(flags, vf, sf)
    print("flags", flags, "vf", vf, "sf", sf, flush=True)
    op = Operator(c.cfg, c.mesh, species=c.species)
    ref = op.rhs(c.u0)
    s = dgx.Solver(c)
    u = to_dev(c.u0)
    got = to_host(s.rhs(u))
    Tg = torch.empty(c.u0.shape[1:], dtype=torch.float64, device="cuda")
    dgx.dgx_thermo(s.ctx, u, Tg)
    s.check()
    s.close()
    e = parity_err(got, ref, flux_scale(op, c.u0))
    eT = np.max(np.abs(to_host(Tg) - T) / T)
    print("parity %.3e, T %.3e" % (e, eT))
    assert e < 1e-11 and eT < 1e-12
