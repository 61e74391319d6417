"""Block CG around the column counts at which its Gram kernel takes other tiles (16, 32, 64).

Reference: the independent CGs of the same operator, which form no Gram
matrix.  Both end at a relative residual of 1e-8, so the currents agree to
1e-8 times the condition of the recovery, held to the 1e-5 of the dense
oracle's comparison.  Two rows per workgroup leave every chunk short.
"""
import numpy as np
import pytest

import synth

from ._meshes import rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nrhs", [2, 15, 16, 17, 32, 33, 64])
def test_block_cg_equals_independent_cgs(nrhs):
    import torch
    import paper_1803_08333_amd as rf
    mesh = rf.Mesh(*synth.icosphere(2))
    start = torch.from_numpy(synth.complex_start(mesh.N, 11)).cuda()
    kh, pol = synth.plane_waves(nrhs, 4)
    j = []
    for block in (0, 1):
        op = rf.Operator(mesh, 1.0, power_start=start, precision=0, block_cg=block)
        x, _, info = op.solve(op.rhs_planewave(np.asarray(kh), np.asarray(pol)), tol=1e-8, maxit=500)
        j.append(x.cpu().numpy())
        op.close()
    assert rel(j[1], j[0]) < 1e-5
    mesh.close()
