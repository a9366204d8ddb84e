"""The gauge action at the edges of its workgroups (half volumes below, at and
past a multiple of 64), on lattices with extents 2, Symanzik and Wilson,
against the oracle.  Tolerance 1e-12 relative: at most 18 x 1200 terms of order
one, each with a rounding error of a few 1e-16."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("L", [(2, 2, 2, 2), (2, 4, 2, 6), (4, 4, 4, 2), (6, 2, 4, 6),
                               (10, 6, 4, 2), (6, 4, 10, 4)])
@pytest.mark.parametrize("c1", [-1.0 / 12.0, 0.0, -0.331])
def test_gauge_action_vs_oracle(L, c1):
    import paper_1801_01473_amd as lq
    g = lq.Geometry(L)
    U = synth.links_haar(L, 551)
    U64 = lq.pack_links(g, torch.from_numpy(np.ascontiguousarray(U)).to("cuda"))
    S, ref = lq.gauge_action(g, U64, 1.9, c1), oracle.gauge_action(L, U, 1.9, c1)
    assert abs(S - ref) <= 1e-12 * abs(ref)
