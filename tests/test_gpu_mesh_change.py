"""A context that changes its octree mesh: coarse, refined, coarse, finer (its
buffers kept, grown and kept again) against a fresh context for each mesh, and
the octree's metric terms (one cell per level) against those of the nodal
coordinates.  N = 3 takes affine kernels, N = 4 the curved ones on the uniform
mesh.  Bound of the coordinates' comparison: 1e-11 of the flux scale, as for
every right-hand side; a fresh context gives the same bits."""
import numpy as np
import pytest

from oracle import amr
from oracle.dgsem import Operator
from paper_2511_17551_amd import workloads as W
from tests.helpers import flux_scale, parity_err, to_dev, to_host

pytestmark = pytest.mark.gpu


def leaves_of(base, centre, radius):
    order = amr.morton_order(base, [(0, i, j, k) for k in range(base) for j in range(base) for i in range(base)])
    if radius == 0.0:
        return order
    mid = (np.array([c[1:] for c in order]) + 0.5) / base
    near = np.linalg.norm(mid - centre, axis=1) < radius
    new, _ = amr.adapt(base, order, {c: int(t) for c, t in zip(order, near)})
    return amr.morton_order(base, new)


@pytest.mark.parametrize("N", [3, 4])
def test_mesh_sequence(N):
    import torch
    from paper_2511_17551_amd import dgx
    assert torch.cuda.is_available()
    cfg = W.base_cfg(3, N, W.EQ_EULER)
    kept = dgx.dgx_create(cfg, None, None)
    for base, radius in ((4, 0.0), (4, 0.4), (4, 0.0), (6, 0.3), (3, 0.0)):
        leaves = leaves_of(base, (0.4, 0.5, 0.6), radius)
        x, faces, mortars, level = amr.mesh(base, N, leaves)
        mesh = W.Mesh(3, N, x, faces, np.zeros((0, 3), np.int32), mortars, np.zeros(0, np.int32), np.zeros((0, 5)),
                      level=level)
        u0 = W.blob_state(x)
        print("N", N, "base", base, "leaves", len(leaves), flush=True)
        res = []
        for ctx, octree in ((kept, True), (None, True), (None, False)):
            h = ctx or dgx.dgx_create(cfg, None, None)
            if octree:
                dgx.dgx_set_octree(h, base, np.asarray(leaves, np.int32))
            else:
                dgx.dgx_set_mesh(h, mesh)
            u = to_dev(u0)
            du = torch.empty_like(u)
            dgx.dgx_rhs(h, u, 0.0, du)
            dgx.dgx_ssprk3_step(h, u, 0.0, 1e-4, 2)
            res.append((to_host(du), to_host(u)))
            dgx.dgx_check(h)
            if ctx is None:
                dgx.dgx_destroy(h)
        assert np.array_equal(res[0][0], res[1][0]) and np.array_equal(res[0][1], res[1][1])
        op = Operator(cfg, mesh)
        scale = flux_scale(op, u0)
        e = max(parity_err(res[0][0], r, scale) for r in (res[2][0], op.rhs(u0)))
        print("parity %.3e" % e)
        assert e < 1e-11
    dgx.dgx_destroy(kept)
