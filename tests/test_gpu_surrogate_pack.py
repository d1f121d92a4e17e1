"""The packed weights that dgx_surrogate_set writes are those that training
keeps up to date: a network trained here, read and set into another context,
predicts and differentiates with the same bits (inference reads the forward
fragments, the gradient the transposed ones too)."""
import numpy as np
import pytest

from oracle.thermo import Mixture
from paper_2511_17551_amd import workloads as W
from tests.helpers import to_dev, to_host

pytestmark = pytest.mark.gpu


def test_set_packs_as_training():
    import torch
    from paper_2511_17551_amd import dgx
    assert torch.cuda.is_available()
    mix = Mixture(W.Species())
    c = W.case_c4(lambda rs, T: mix.rho_e(rs, T), lambda rs, T: mix.rho_cv(rs, T), nr=4, nth=8)
    rs, T = W.far_chem_states(1000, seed=8)
    v = np.random.default_rng(8).uniform(-1000.0, 1000.0, (2, 1000))
    rho = rs.sum(0)
    st = to_dev(np.concatenate([rs, rho * v, (mix.rho_e(rs, T) + 0.5 * rho * (v * v).sum(0))[None]]))
    Td = to_dev(T)
    a, b = dgx.Solver(c), dgx.Solver(c)
    dgx.dgx_surrogate_init(a.ctx, st, Td)
    dgx.dgx_surrogate_train(a.ctx, st, Td, 2, 128, 1e-2)
    prm = dgx.dgx_surrogate_get(a.ctx)
    dgx.dgx_surrogate_set(b.ctx, np.zeros_like(prm))
    dgx.dgx_surrogate_set(b.ctx, prm)
    assert np.array_equal(dgx.dgx_surrogate_get(b.ctx), prm)
    out = []
    for s in (a, b):
        Tg = torch.empty_like(Td)
        dgx.dgx_surrogate_predict(s.ctx, st, Tg)
        g, loss = dgx.dgx_surrogate_grad(s.ctx, st, Td)
        out.append((to_host(Tg), g, loss))
        s.close()
    assert np.isfinite(out[0][0]).all() and np.abs(out[0][1]).max() > 0
    for x, y in zip(*out):
        assert np.array_equal(x, y)
