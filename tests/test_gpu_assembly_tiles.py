"""The dense blocks at the edges of the assembly's tiles (512, 1024 and 2048
edges, the last one ragged; one tile alone; 64-edge tiles with few edges left):
sampled rows of T_A and V against the oracle's, exact symmetry, and V written
for every pair of cells.  Far pairs are FP32 sums of 49 terms on both cells,
stored in complex64: 2e-6, as for the other block tests."""
import numpy as np
import pytest

import synth
from oracle import assembly
from oracle.topology import Topology

from ._meshes import rel

pytestmark = pytest.mark.gpu

# N = 162, 450, 513, 1092, 1920, 6168 (the second size above 6144 edges is 7680, in the full-size tests)
MESHES = {"cube3": lambda: synth.cube(3), "cube5": lambda: synth.cube(5), "torus19x9": lambda: synth.torus(19, 9, seed=2),
          "torus28x13": lambda: synth.torus(28, 13, seed=2), "ico3": lambda: synth.icosphere(3),
          "torus257x8": lambda: synth.torus(257, 8, seed=2)}


@pytest.mark.parametrize("name", sorted(MESHES))
def test_block_rows(name):
    import paper_1803_08333_amd as rf
    xyz, tri = MESHES[name]()
    top, k = Topology(xyz, tri), 1.1
    m = rf.Mesh(xyz, tri)
    op = rf.Operator(m, k, scaling=1)
    TA, V = (t.cpu().numpy() for t in op.export())
    assert np.array_equal(TA, TA.T) and np.array_equal(V, V.T)
    assert np.all(np.isfinite(TA)) and np.all(V != 0)
    rng = np.random.default_rng(4)
    edges = np.unique(np.concatenate([[0, 63, 64, top.N - 1], rng.integers(0, top.N, 8)]) % top.N)
    assert rel(TA[edges], assembly.ta_rows(top, k, edges)) < 2e-6
    cells = np.unique(np.concatenate([[0, top.C - 1], rng.integers(0, top.C, 6)]))
    assert rel(V[cells], assembly.block_rows(top, k, cells)[0]) < 2e-6
    op.close()
    m.close()


@pytest.mark.parametrize("name", ["ico3", "torus28x13", "ico4"])
def test_block_rows_of_shuffled_cells(name):
    """Cells in random order: an edge's two cells lie anywhere in its tile, so
    that pairs whose first cell has the higher index are taken in every tile."""
    import paper_1803_08333_amd as rf
    xyz, tri = synth.icosphere(4) if name == "ico4" else MESHES[name]()
    tri = np.ascontiguousarray(tri[np.random.default_rng(7).permutation(len(tri))])
    top, k = Topology(xyz, tri), 1.1
    m = rf.Mesh(xyz, tri)
    op = rf.Operator(m, k, scaling=1)
    TA, V = (t.cpu().numpy() for t in op.export())
    assert np.array_equal(TA, TA.T) and np.array_equal(V, V.T)
    rng = np.random.default_rng(4)
    edges = np.unique(np.concatenate([[0, 63, 64, top.N - 1], rng.integers(0, top.N, 6)]))
    assert rel(TA[edges], assembly.ta_rows(top, k, edges)) < 2e-6
    cells = np.unique(np.concatenate([[0, top.C - 1], rng.integers(0, top.C, 4)]))
    assert rel(V[cells], assembly.block_rows(top, k, cells)[0]) < 2e-6
    op.close()
    m.close()
