"""The compressed blocks do not depend on timing: every thread of a block's
adaptive cross approximation divides its row by the same pivot.  Two operators
of one mesh are equal bit for bit, and both stay within the tolerance's bound of
the dense blocks (10 x tol, as for the oracle's compressed blocks)."""
import numpy as np
import pytest

import synth

from ._meshes import rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tol", [1e-3, 1e-4])
def test_compressed_blocks_repeat(tol):
    import paper_1803_08333_amd as rf
    m = rf.Mesh(*synth.icosphere(4))
    dense = rf.Operator(m, 1.0, scaling=1)
    ref = [t.cpu().numpy() for t in dense.export()]
    dense.close()
    got = []
    for _ in range(3):
        op = rf.Operator(m, 1.0, scaling=1, aca_tol=tol)
        got.append([t.cpu().numpy() for t in op.export()])
        op.close()
    for blocks in got:
        for a, b, r in zip(blocks, got[0], ref):
            assert np.array_equal(a, b)
            assert rel(a, r) < 10 * tol
    m.close()
