"""The fermion force on both sides of the rule that splits the pairs of a workgroup.

Half volumes 16384 (the largest with two groups) and 16416 (one group, the last
workgroup half empty), even and odd numbers of pairs.  The bound is that of the
other force tests: chains of at most 27 + npair additions of terms whose absolute
sum exceeds the largest element by less than 100.
"""
import numpy as np
import pytest

import oracle
import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("L", [(16, 16, 16, 8), (2, 4, 4, 1026)])
@pytest.mark.parametrize("npf,ns", [(2, 2), (1, 5)])
@pytest.mark.parametrize("mode", [0, 1])
def test_force_pair_groups(L, npf, ns, mode):
    import paper_1801_01473_amd as lq

    g = lq.Geometry(L)
    U = synth.links_haar(L, 321)
    X = synth.gaussian_even_source(L, npf * ns, 322).reshape(npf, ns, -1, 3)
    al = np.linspace(0.4, 2.1, ns)
    cu = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")  # noqa: E731
    Xp = lq.pack_spinor(g, cu(X.reshape(-1, g.V, 3)), 0)
    U64 = lq.pack_links(g, cu(U))
    F = lq.fermion_force(g, U64, al, Xp, mode=mode)
    ref = oracle.force(L, U, al, X, mode=mode)
    assert H.max_rel(lq.unpack_links(g, F).cpu().numpy(), ref) <= 1e-12
    F2 = lq.fermion_force(g, U64, al, Xp, mode=mode, out=F.clone(), accumulate=True)
    assert torch.equal(F2, 2 * F)
