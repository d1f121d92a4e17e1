"""The chemistry step's three kernels (grouped rates; reaction by reaction with
the molecules first; reaction by reaction with other molecule flags) against
the oracle, in 2D and 3D: species within 1e-11 rho (the bound of the chemistry
tests) and the same numbers of substeps, at a step that moves them."""
import numpy as np
import pytest

from oracle.chemistry import backward_euler
from oracle.kinetics import Kinetics
from oracle.thermo import Mixture
from paper_2511_17551_amd import workloads as W
from tests.helpers import to_dev, to_host
from tests.test_gpu_chem import dgx  # noqa: F401
from tests.test_gpu_chem_groups import mechanism

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("kernel", ["grouped", "general", "other_flags"])
def test_kernels(dgx, dim, kernel):  # noqa: F811
    sp = W.Species()
    if kernel == "other_flags":  # O2 without internal modes
        sp = W.Species(molecule=np.array([1, 0, 1, 0, 0], np.int32), theta_v=np.array([3393.0, 0.0, 2739.0, 0.0, 0.0]))
    mix = Mixture(sp)
    energy = lambda rs, T: mix.rho_e(rs, T)  # noqa: E731
    if dim == 2:
        c = W.case_c4(energy, lambda rs, T: mix.rho_cv(rs, T), nr=4, nth=8, hot=True)
        c.cfg = dict(c.cfg, eq=W.EQ_EULER_MIX)
    else:
        c = W.curved_periodic_mixture_case(energy, n=2, N=4, T0=6000.0)
    c.species = sp
    c.reactions = mechanism("two_partners" if kernel == "general" else "shuffled")
    print("kernel", kernel, "dim", dim, flush=True)
    dt = 1e-9
    flat = c.u0.reshape(c.u0.shape[0], -1)
    rho = flat[:5].sum(0)
    rhoe = flat[5 + dim] - 0.5 * (flat[5:5 + dim] ** 2).sum(0) / rho
    T0, _ = mix.solve_T(flat[:5], rhoe, c.cfg["T_guess"])
    ref, _, it, nsub = backward_euler(mix, Kinetics(sp, c.reactions), flat[:5], rhoe, dt, T0)
    s = dgx.Solver(c)
    u = to_dev(c.u0)
    st = dgx.dgx_chem_step(s.ctx, u, dt)
    s.check()
    got = to_host(u).reshape(flat.shape)
    s.close()
    err = np.max(np.abs(got[:5] - ref) / rho)
    moved = np.max(np.abs(ref - flat[:5]) / rho)
    print("err %.3e moved %.3e iters %d / oracle %d" % (err, moved, st["iters_max"], it.max()))
    assert st["nonconverged"] == 0 and st["substeps_total"] == nsub.sum()
    assert moved > 1e-7 and err < 1e-11
    assert np.array_equal(got[5:], flat[5:])
