"""The far field at the edges of its tiles: directions around the groups of 16
and beyond one launch's chunk (16 384), right-hand sides around the column
groups (2, 5, 10, 21), plain and split, against the oracle.  Both sides sum
7 C terms of one size in FP64 in different orders: 1e-12, as for the far field
itself."""
import numpy as np
import pytest

import synth
from oracle import farfield
from oracle.topology import Topology

from ._meshes import rel

pytestmark = pytest.mark.gpu


def _dirs(n, seed):
    d = np.random.default_rng(seed).normal(size=(n, 3))
    return d / np.linalg.norm(d, axis=1, keepdims=True)


@pytest.mark.parametrize("nrhs,ndir", [(1, 1), (2, 15), (3, 16), (5, 17), (6, 33), (10, 2), (11, 31), (21, 48), (22, 5),
                                       (43, 16), (2, 16384 + 19)])
@pytest.mark.parametrize("split", [False, True])
def test_far_field_tiles(nrhs, ndir, split):
    import torch
    import paper_1803_08333_amd as rf
    xyz, tri = synth.icosphere(1) if ndir > 1000 else synth.torus(9, 7, seed=1)
    top, k = Topology(xyz, tri), 0.8
    m = rf.Mesh(xyz, tri)
    op = rf.Operator(m, k, scaling=1)
    rng = np.random.default_rng(nrhs)
    j, js = (rng.normal(size=(nrhs, top.N)) + 1j * rng.normal(size=(nrhs, top.N)) for _ in range(2))
    d = _dirs(ndir, 1)
    if split:
        # the split form of any pair: (exp(-it) - 1) on the first, exp(-it) on the second
        F, s = op.far_field_split(torch.from_numpy(j).cuda(), torch.from_numpy(js).cuda(), d)
        ref = farfield.far_field(top, k, j, d) - farfield.far_field(top, 0.0, j, d) + farfield.far_field(top, k, js, d)
    else:
        F, s = op.far_field(torch.from_numpy(j).cuda(), d)
        ref = farfield.far_field(top, k, j, d)
    assert rel(F.cpu().numpy(), ref) < 1e-12
    sref = farfield.rcs(k, ref, d)
    assert np.abs(s.cpu().numpy() - sref).max() <= 1e-11 * sref.max()
    op.close()
    m.close()
