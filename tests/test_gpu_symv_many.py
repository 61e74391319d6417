"""Products with three or more right-hand sides at the edges of the symmetric kernels' blocks.

The kernel that takes three to eight right-hand sides keeps every chain of sums
of the one that takes a single right-hand side, so each column has to be the
same bits with any number of others beside it.  Sizes fall around the 128 and
256 blocks and their 32-row stages; inputs go through each fused gather (the
projections, the operator with its paired products).  The single product
itself is held to dense FP64 products (a sum of n <= 10800 terms:
100 sqrt(n) 2^-53 = 1.2e-12).
"""
import numpy as np
import pytest

import synth

from ._meshes import rel

pytestmark = pytest.mark.gpu

# (N, C, V): (30, 20, 12), (162, 108, 56), (384, 256, 130), (399, 266, 133), (2352, 1568, 784), (10800, 7200, 3600)
MESHES = {"ico0": lambda: synth.icosphere(0), "cube3": lambda: synth.cube(3), "torus16x8": lambda: synth.torus(16, 8, seed=2),
          "torus19x7": lambda: synth.torus(19, 7, seed=2), "torus28x28": lambda: synth.torus(28, 28, seed=2),
          "torus60x60": lambda: synth.torus(60, 60, seed=2)}


@pytest.mark.parametrize("name", sorted(MESHES))
def test_columns_do_not_depend_on_their_number(name):
    import torch
    import paper_1803_08333_amd as rf
    mesh = rf.Mesh(*MESHES[name]())
    rng = np.random.default_rng(5)
    gpu = lambda *s: torch.from_numpy(rng.normal(size=s) + 1j * rng.normal(size=s)).cuda()  # noqa: E731
    for star in (0, 1):
        op = rf.Operator(mesh, 0.9, scaling=1, outer_star=star)
        x = gpu(17, mesh.N)
        one = torch.cat([op.apply(x[i:i + 1]) for i in range(7)])
        for nr in (3, 4, 7):
            assert torch.equal(op.apply(x[:nr]), one[:nr])
        if star:
            for which in (rf.PROJ_SIGMA, rf.PROJ_LH, rf.PROJ_LPINV, rf.PROJ_GLL_INV):
                z = gpu(17, {rf.PROJ_LPINV: mesh.C, rf.PROJ_GLL_INV: mesh.V}.get(which, mesh.N))
                one = torch.cat([op.project(which, z[i:i + 1]) for i in range(17)])
                for nr in (2, 3, 5, 8, 9, 11, 17):
                    assert torch.equal(op.project(which, z[:nr]), one[:nr])
        else:
            for which, M in enumerate(op.export()):
                z = gpu(7, len(M))
                for conj in (False, True):
                    one = torch.cat([op.matvec(which, z[i:i + 1], conj=conj) for i in range(7)])
                    for nr in (3, 5, 7):
                        assert torch.equal(op.matvec(which, z[:nr], conj=conj), one[:nr])
                    y = z[:2].cpu().numpy() @ (M.conj() if conj else M).cpu().numpy().astype(np.complex128)
                    assert rel(one[:2].cpu().numpy(), y) < 1.2e-12
        op.close()
    mesh.close()
