"""The fermion force at the edges of its 64-site workgroups and of its pair loop.

Each element is a sum of 3 (terms of U M) x 3 npair x 24 (terms of chi) products
taken in chains of at most 24 + npair + 3 additions, so its error is below
(27 + npair) * 1.1e-16 < 1e-14 of the sum of the absolute terms, which for
Gaussian X exceeds the largest element by less than 100: 1e-12 bounds it.
"""
import numpy as np
import pytest

import oracle
import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# half volumes 8 (one partial workgroup), 64 (one full), 72, 1080 (17, the last
# with 56 sites, tiled) and 1 to 3 pairs (first, even and odd passes of the loop)
@pytest.mark.parametrize("L", [(2, 2, 2, 2), (4, 4, 4, 2), (6, 2, 6, 2), (6, 6, 6, 10)])
@pytest.mark.parametrize("npf,ns", [(1, 1), (1, 2), (3, 1)])
def test_force_workgroup_and_pair_edges(L, npf, ns):
    import paper_1801_01473_amd as lq

    g = lq.Geometry(L)
    U = synth.links_haar(L, 311)
    X = synth.gaussian_even_source(L, npf * ns, 312).reshape(npf, ns, -1, 3)
    al = np.array([0.7, 1.9])[:ns]
    cu = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")  # noqa: E731
    Xp = lq.pack_spinor(g, cu(X.reshape(-1, g.V, 3)), 0)
    F = lq.fermion_force(g, lq.pack_links(g, cu(U)), al, Xp)
    got = lq.unpack_links(g, F).cpu().numpy()
    assert H.max_rel(got, oracle.force(L, U, al, X)) <= 1e-12
