"""The far field of a current does not depend on the call it is part of, and
every width of the sums' workgroups is used and right.

Bits: the order of a current's sums follows from the body alone, so a call with
other currents or other directions beside it returns the same bits.  Against the
oracle both sides sum 7 C terms of one size in FP64 in different orders: 1e-12,
as for the far field itself."""
import numpy as np
import pytest

import synth
from oracle import farfield
from oracle.topology import Topology

from ._meshes import rel

pytestmark = pytest.mark.gpu

MESHES = {"ico1": lambda: synth.icosphere(1), "torus9x7": lambda: synth.torus(9, 7, seed=1), "cube9": lambda: synth.cube(9)}


def _dirs(n, seed):
    d = np.random.default_rng(seed).normal(size=(n, 3))
    return d / np.linalg.norm(d, axis=1, keepdims=True)


def _currents(nrhs, N, seed):
    import torch
    rng = np.random.default_rng(seed)
    return [torch.from_numpy(rng.normal(size=(nrhs, N)) + 1j * rng.normal(size=(nrhs, N))).cuda() for _ in range(2)]


def _call(op, split, j, js, d):
    return op.far_field_split(j, js, d) if split else op.far_field(j, d)


@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("name", sorted(MESHES))
def test_far_field_does_not_depend_on_the_batch(name, split):
    import torch
    import paper_1803_08333_amd as rf
    m = rf.Mesh(*MESHES[name]())
    op = rf.Operator(m, 0.8, scaling=1)
    j, js = _currents(37, m.N, 3)
    d = _dirs(600, 4)
    F, s = _call(op, split, j, js, d)
    for r0, r1, d0, d1 in ((0, 1, 0, 600), (36, 37, 5, 6), (0, 5, 17, 60), (3, 11, 0, 17), (2, 18, 100, 300),
                           (5, 26, 0, 600), (0, 37, 599, 600)):
        f, t = _call(op, split, j[r0:r1], js[r0:r1], d[d0:d1])
        assert torch.equal(f, F[r0:r1, d0:d1]) and torch.equal(t, s[r0:r1, d0:d1])
    op.close()
    m.close()


# 6 nrhs columns fill 1 to 8 groups of 16 and leave a group short, or take 2 workgroups of them; 600 directions of a body of
# 126 cells are enough workgroups for the width to be the number of groups
@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("nrhs,width", [(1, 1), (2, 1), (5, 2), (7, 3), (10, 4), (13, 5), (15, 6), (18, 7), (21, 8), (42, 8)])
def test_far_field_of_every_width(nrhs, width, split):
    import paper_1803_08333_amd as rf
    xyz, tri = MESHES["torus9x7"]()
    top, k = Topology(xyz, tri), 0.8
    m = rf.Mesh(xyz, tri)
    op = rf.Operator(m, k, scaling=1)
    j, js = _currents(nrhs, m.N, nrhs)
    d = _dirs(600, 1)
    rf.profile_enable(True)
    try:
        F, s = _call(op, split, j, js, d)
        assert rf.profile_read(f"farfield_w{width}")[1] == 1
    finally:
        rf.profile_enable(False)
    j, js = j.cpu().numpy(), js.cpu().numpy()
    ref = farfield.far_field(top, k, j, d)
    if split:  # (exp(-it) - 1) on the first part, exp(-it) on the second
        ref = ref - farfield.far_field(top, 0.0, j, d) + farfield.far_field(top, k, js, d)
    assert rel(F.cpu().numpy(), ref) < 1e-12
    sref = farfield.rcs(k, ref, d)
    assert np.abs(s.cpu().numpy() - sref).max() <= 1e-11 * sref.max()
    op.close()
    m.close()


@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("k", [5.0, 40.0, 3e4, 2e5])
def test_far_field_of_large_phases(k, split):
    """Phases k dhat . x of every quadrant, of thousands of turns, and on both
    sides of 1e5, from where another sine is taken.  Each side rounds a phase by
    at most 4 x 2^-53 k: 1e-12 + 2e-15 k."""
    import paper_1803_08333_amd as rf
    xyz, tri = synth.icosphere(2)
    top = Topology(xyz, tri)
    m = rf.Mesh(xyz, tri)
    op = rf.Operator(m, k, scaling=1)
    j, js = _currents(3, m.N, 5)
    d = _dirs(40, 2)
    F, s = _call(op, split, j, js, d)
    j, js = j.cpu().numpy(), js.cpu().numpy()
    ref = farfield.far_field(top, k, j, d)
    if split:
        ref = ref - farfield.far_field(top, 0.0, j, d) + farfield.far_field(top, k, js, d)
    tol = 1e-12 + 2e-15 * k
    assert rel(F.cpu().numpy(), ref) < tol
    sref = farfield.rcs(k, ref, d)
    assert np.abs(s.cpu().numpy() - sref).max() <= 10 * tol * sref.max()
    op.close()
    m.close()
