"""Device memory that calls take: what an operator never uses it does not hold,
and a call that a larger scratch only makes faster still runs without it.

The allocator registered here is torch's, counted or refusing blocks above a
size."""
import contextlib

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@contextlib.contextmanager
def _allocator(limit=None):
    """torch's allocator, refusing blocks above `limit` bytes; yields the live blocks and the refused sizes."""
    import torch
    import paper_1803_08333_amd as rf
    live, refused = {}, []

    def alloc(nbytes):
        if limit is not None and nbytes > limit:
            refused.append(nbytes)
            return None
        p = torch.cuda.caching_allocator_alloc(nbytes)
        live[p] = nbytes
        return p

    def free(p, nbytes):
        del live[p]
        torch.cuda.caching_allocator_delete(p)

    rf.set_allocator(alloc, free)
    try:
        yield live, refused
    finally:
        rf.use_torch_allocator()


def test_compressed_operator_holds_no_dense_scratch():
    """A compressed operator with sparse projectors runs no dense product: it
    holds its stored entries and O(N) beside them (workspace for four right-hand
    sides 2 KB an edge, near pairs 1.5 KB, projections, factors: below 8 KB an
    edge in all), where the slots of dense products would be 24 KB an edge."""
    import paper_1803_08333_amd as rf
    with _allocator() as (live, _):
        m = rf.Mesh(*synth.icosphere(5))
        op = rf.Operator(m, 1.0, scaling=1, aca_tol=1e-2)
        c = op.compression()
        stored = 8 * (sum(c["dense_entries"]) + sum(c["lowrank_entries"]))
        assert sum(live.values()) < stored + 8192 * m.N, (sum(live.values()) - stored) / m.N
        op.close()
        m.close()
        assert not live
