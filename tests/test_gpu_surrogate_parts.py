"""The gradient's split into 16-sample tiles, groups of four tiles and parts
of 1,024 tiles, at the edges of each: against the oracle, with the bounds of
test_gpu_surrogate.py (whose fixtures it shares)."""
import numpy as np
import pytest

from oracle import mlp
from tests.helpers import to_dev
from tests.test_gpu_surrogate import dgx, solver, state_set  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [15, 65, 16384, 16384 + 53])
def test_gradient_parts(dgx, solver, count):  # noqa: F811
    u, T = state_set(count, 2)
    ud, Td = to_dev(u), to_dev(T)
    print("count", count, flush=True)
    dgx.dgx_surrogate_init(solver.ctx, ud, Td, seed=7)
    prm = dgx.dgx_surrogate_get(solver.ctx)
    g, loss = dgx.dgx_surrogate_grad(solver.ctx, ud, Td)
    p = mlp.unpack(prm.astype(np.float64))
    raw = mlp.raw_features(u[:5], u[7] - 0.5 * (u[5] ** 2 + u[6] ** 2) / u[:5].sum(0))
    lo, go = mlp.loss_and_grad(p, mlp.standardise(raw, p), (T - p["Tm"]) / p["Ts"])
    gp = mlp.unpack(np.concatenate([g.astype(np.float64), np.zeros(14)]))
    assert abs(loss - lo) < 1e-3 * lo
    for name, _ in mlp.SIZES:
        rel = np.linalg.norm(gp[name] - go[name]) / np.linalg.norm(go[name])
        print("grad %s rel L2 %.3e" % (name, rel))
        assert rel < 5e-3, name
    # one training step leaves the weights' packed copy equal to the weights:
    # setting the same parameters again (packed on the host) gives the same gradient
    dgx.dgx_surrogate_train(solver.ctx, *[to_dev(a) for a in state_set(320, 5)], epochs=1, batch=192, lr=2e-3)
    g1, _ = dgx.dgx_surrogate_grad(solver.ctx, ud, Td)
    dgx.dgx_surrogate_set(solver.ctx, dgx.dgx_surrogate_get(solver.ctx))
    g2, _ = dgx.dgx_surrogate_grad(solver.ctx, ud, Td)
    assert np.array_equal(g1, g2)
