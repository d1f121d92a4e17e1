"""The chemistry step's two rate evaluations (reactions grouped by net
stoichiometry, and reaction by reaction) against the oracle on mechanisms at
the edges of the rule that chooses between them, and on cold gas, where the
rate constants leave the exponent range."""
import numpy as np
import pytest

from paper_2511_17551_amd import workloads as W
from tests.helpers import to_dev, to_host
from tests.test_gpu_chem import dgx, frozen_case, oracle_chem, thermo_fns  # noqa: F401

pytestmark = pytest.mark.gpu


def take(rx, rows):
    return W.Reactions(rx.A[rows], rx.b[rows], rx.theta_a[rows], rx.nu[rows], rx.nup[rows])


def add(rx, nu, nup, A, b, th):
    row = lambda v: np.array([v], np.int32)  # noqa: E731
    return W.Reactions(np.append(rx.A, A), np.append(rx.b, b), np.append(rx.theta_a, th),
                       np.concatenate([rx.nu, row(nu)]), np.concatenate([rx.nup, row(nup)]))


def mechanism(kind):
    rx = W.park17_reactions(4)
    if kind == "shuffled":        # partners of a group out of order
        return take(rx, np.random.default_rng(1).permutation(17))
    if kind == "partial":         # groups with some partners missing
        return take(rx, np.array([0, 3, 6, 9, 11, 16]))
    if kind == "repeated":        # the same reaction twice: a second group
        return take(rx, np.array([0, 1, 2, 0, 5, 15, 15]))
    if kind == "no_partner":      # N2 <-> 2 N beside the dissociations with partners
        return add(rx, [1, 0, 0, 0, 0], [0, 0, 0, 2, 0], 1e6, -0.5, 113200.0)
    if kind == "two_partners":    # N2 + N + O <-> 3 N + O: reaction by reaction
        return add(rx, [1, 0, 0, 1, 1], [0, 0, 0, 3, 1], 1e8, -0.5, 113200.0)
    # O2 + 2 N <-> 2 NO: three reactant factors, reaction by reaction
    return add(rx, [0, 1, 0, 2, 0], [0, 0, 2, 0, 0], 1e6, -0.5, 1000.0)


@pytest.mark.parametrize("kind", ["shuffled", "partial", "repeated", "no_partner", "two_partners", "three_factors"])
def test_mechanisms(dgx, thermo_fns, kind):  # noqa: F811
    """Species within 1e-11 rho of the oracle (the bound of the chemistry tests) at a step that moves them."""
    c = frozen_case(thermo_fns, 4, 8)
    c.reactions = mechanism(kind)
    print("mechanism", kind, flush=True)
    dt = 1e-9
    ref, _, it, nsub = oracle_chem(c, c.u0, dt)
    s = dgx.Solver(c)
    u = to_dev(c.u0)
    st = dgx.dgx_chem_step(s.ctx, u, dt)
    s.check()
    got = to_host(u)
    s.close()
    rho = c.u0[:5].sum(0)
    err = np.max(np.abs(got[:5] - ref[:5]) / rho)
    moved = np.max(np.abs(ref[:5] - c.u0[:5]) / rho)
    print("err %.3e moved %.3e iters %d / oracle %d" % (err, moved, st["iters_max"], it.max()))
    assert st["nonconverged"] == 0 and st["substeps_total"] == nsub.sum()
    assert moved > 1e-6 and err < 1e-11


def test_cold_gas(dgx, thermo_fns):  # noqa: F811
    """25-400 K with atoms present (ln k_f down to -4500, ln K_c likewise), and molecules alone at 1e-4 K."""
    c = frozen_case(thermo_fns, 4, 8)
    rng = np.random.default_rng(3)
    shape = c.u0.shape[1:]
    T = 10.0 ** rng.uniform(np.log10(25.0), np.log10(400.0), shape)
    Y = np.stack([np.full(shape, 0.76), np.full(shape, 0.23)] + [10.0 ** rng.uniform(-12, -4, shape) for _ in range(3)])
    Y[2:, :4] = 0.0
    T[:4] = 1e-4
    Y = Y / Y.sum(0)
    rho = 10.0 ** rng.uniform(-4, 0, shape)
    u0 = c.u0.copy()
    u0[:5] = Y * rho
    u0[5:7] = 0.0
    u0[7] = thermo_fns[0]((Y * rho).reshape(5, -1), T.reshape(-1)).reshape(shape)
    print("cold gas", flush=True)
    dt = 1e-7
    ref, _, it, nsub = oracle_chem(c, u0, dt)
    s = dgx.Solver(c)
    u = to_dev(u0)
    st = dgx.dgx_chem_step(s.ctx, u, dt)
    s.check()
    got = to_host(u)
    s.close()
    err = np.max(np.abs(got[:5] - ref[:5]) / rho)
    moved = np.max(np.abs(ref[:5] - u0[:5]) / rho)
    print("err %.3e moved %.3e substeps %d / oracle %d" % (err, moved, st["substeps_total"], nsub.sum()))
    assert st["nonconverged"] == 0 and np.isfinite(got).all()
    assert err < 1e-11
    assert np.array_equal(got[:5, :4], u0[:5, :4])
