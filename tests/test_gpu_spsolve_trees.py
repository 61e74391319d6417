"""Sparse projector solves on bodies whose dissection leaves parts that no
separator's row reaches: such a part hangs below a later supernode than the
columns around it, and belongs to one subtree of the solve only.  Cubes and tori
at these attitudes have one to eight of them in L or G_ll.

Reference: the defining equations, L (L^+ x) = x - mean x and G_ll (G_ll^-1 x)
= x, to 1e-11 (the condition of L at this size, about 1e5, times 2^-53, with a
factor of 1000), and the same bits from a second call."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _attitude(xyz, seed):
    q, r = np.linalg.qr(np.random.default_rng(seed).normal(size=(3, 3)))
    q = q * np.sign(np.diag(r))
    q[:, 0] *= np.sign(np.linalg.det(q))
    return np.ascontiguousarray(xyz @ q.T)


@pytest.mark.parametrize("name,seed", [("cube33", 0), ("cube33", 1), ("cube33", 2), ("cube33", 4), ("torus81x81", 3),
                                       ("torus81x81", 5)])
def test_sparse_solves_of_uneven_dissections(name, seed):
    import scipy.sparse as sp
    import torch
    import paper_1803_08333_amd as rf
    xyz, tri = synth.torus(81, 81, seed=3) if name == "torus81x81" else synth.cube(33)
    xyz = _attitude(xyz, seed)
    mesh = rf.Mesh(xyz, tri)
    assert mesh.C > 12288
    op = rf.Operator(mesh, 0.5, scaling=1, aca_tol=1e-2)
    C, V = mesh.C, mesh.V
    tri = np.asarray(tri).astype(np.int64)
    key = np.sort(np.stack([tri[:, [1, 2]], tri[:, [2, 0]], tri[:, [0, 1]]], 1).reshape(-1, 2), axis=1)
    _, inv = np.unique(key[:, 0] * V + key[:, 1], return_inverse=True)
    inc = sp.csr_matrix((np.ones(3 * C), (np.repeat(np.arange(C), 3), inv.reshape(-1))))
    lap = 6.0 * sp.identity(C) - inc @ inc.T  # 3 on the diagonal, -1 to each neighbour
    area = np.linalg.norm(np.cross(xyz[tri[:, 1]] - xyz[tri[:, 0]], xyz[tri[:, 2]] - xyz[tri[:, 0]]), axis=1) / 2
    i, j = np.repeat(tri, 3, axis=1).reshape(-1), np.tile(tri, (1, 3)).reshape(-1)
    gll = sp.csr_matrix((np.where(i == j, 1 / 6, 1 / 12) * np.repeat(area, 9), (i, j)), shape=(V, V))
    rng = np.random.default_rng(seed)
    for nrhs in (1, 3, 64):
        for which, n, M in ((rf.PROJ_LPINV, C, lap), (rf.PROJ_GLL_INV, V, gll)):
            x = rng.normal(size=(nrhs, n)) + 1j * rng.normal(size=(nrhs, n))
            xd = torch.from_numpy(x).cuda()
            y, again = op.project(which, xd), op.project(which, xd)
            want = x - x.mean(1, keepdims=True) if which == rf.PROJ_LPINV else x
            assert np.linalg.norm((M @ y.cpu().numpy().T).T - want) < 1e-11 * np.linalg.norm(x)
            assert torch.equal(y, again)
    op.close()
    mesh.close()
