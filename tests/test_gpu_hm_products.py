"""Compressed products at the edges of their operands: right-hand sides around
the groups of 8, a last tile of few edges, tiles that home more or fewer than 16
cells a wave, ranks around 16, plain and conjugated, against complex128 products
of the written-out blocks.  Those are rounded to complex64 once (6e-8 of each
entry): 2e-6, as for the other compressed products."""
import numpy as np
import pytest

import synth

from ._meshes import rel

pytestmark = pytest.mark.gpu

MESHES = {"cube9": lambda: synth.cube(9), "torus61x11": lambda: synth.torus(61, 11, seed=2),
          "graded3": lambda: synth.graded_sphere(3, 0.6)}


@pytest.mark.parametrize("name", sorted(MESHES))
@pytest.mark.parametrize("tol", [1e-2, 1e-4, 1e-6])
def test_compressed_products(name, tol):
    import torch
    import paper_1803_08333_amd as rf
    m = rf.Mesh(*MESHES[name]())
    op = rf.Operator(m, 1.2, scaling=1, aca_tol=tol)
    rng = np.random.default_rng(3)
    for which, M in enumerate(t.cpu().numpy().astype(np.complex128) for t in op.export()):
        for nrhs in (1, 7, 8, 17):
            x = rng.normal(size=(nrhs, len(M))) + 1j * rng.normal(size=(nrhs, len(M)))
            for conj in (False, True):
                y = op.matvec(which, torch.from_numpy(x).cuda(), conj=conj).cpu().numpy()
                assert rel(y, x @ (M.conj() if conj else M)) < 2e-6
    op.close()
    m.close()
