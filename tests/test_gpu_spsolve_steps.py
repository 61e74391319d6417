"""Sparse projector solves at the edges of their steps.

Bodies just beyond the size from which the projectors are factored sparsely, so
that one, some and 16 right-hand sides per workgroup (and a last group that is
not full) meet subtrees of every height.  A right-hand side's sums in a subtree
do not depend on the others.  Reference: the defining equations, L (L^+ x) =
x - mean x and G_ll (G_ll^-1 x) = x, to 1e-11 (the condition of L at this size,
about 1e5, times 2^-53, with a factor of 1000).
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nrhs", [1, 3, 17, 64])
@pytest.mark.parametrize("name", ["torus81x79", "cube33"])
def test_sparse_solves(name, nrhs):
    import scipy.sparse as sp
    import torch
    import paper_1803_08333_amd as rf
    xyz, tri = synth.torus(81, 79, seed=3) if name == "torus81x79" else synth.cube(33)
    mesh = rf.Mesh(xyz, tri)
    assert mesh.C > 12288
    op = rf.Operator(mesh, 0.5, scaling=1, aca_tol=1e-2)
    rng = np.random.default_rng(nrhs)
    C, V = mesh.C, mesh.V
    tri = np.asarray(tri).astype(np.int64)
    key = np.sort(np.stack([tri[:, [1, 2]], tri[:, [2, 0]], tri[:, [0, 1]]], 1).reshape(-1, 2), axis=1)
    _, inv = np.unique(key[:, 0] * V + key[:, 1], return_inverse=True)
    inc = sp.csr_matrix((np.ones(3 * C), (np.repeat(np.arange(C), 3), inv.reshape(-1))))
    lap = 6.0 * sp.identity(C) - inc @ inc.T  # 3 on the diagonal, -1 to each neighbour
    area = np.linalg.norm(np.cross(xyz[tri[:, 1]] - xyz[tri[:, 0]], xyz[tri[:, 2]] - xyz[tri[:, 0]]), axis=1) / 2
    i, j = np.repeat(tri, 3, axis=1).reshape(-1), np.tile(tri, (1, 3)).reshape(-1)
    gll = sp.csr_matrix((np.where(i == j, 1 / 6, 1 / 12) * np.repeat(area, 9), (i, j)), shape=(V, V))
    for which, n, M in ((rf.PROJ_LPINV, C, lap), (rf.PROJ_GLL_INV, V, gll)):
        x = rng.normal(size=(nrhs, n)) + 1j * rng.normal(size=(nrhs, n))
        y = op.project(which, torch.from_numpy(x).cuda()).cpu().numpy()
        want = x - x.mean(1, keepdims=True) if which == rf.PROJ_LPINV else x
        assert np.linalg.norm((M @ y.T).T - want) < 1e-11 * np.linalg.norm(x)
    op.close()
    mesh.close()
