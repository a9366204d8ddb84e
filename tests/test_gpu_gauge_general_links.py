"""The Symanzik force of links that are not unitary to rounding.

Moving a loop along a link V takes V^dag for V^-1, so the loop fields alone lose
accuracy in first order of V^dag V - 1; links that are off by more than rounding
must get their staples multiplied out.  Against the oracle, which enumerates the
loops and holds for any matrices: single-precision links (1e-7 off), noisy ones
(1e-4), Gaussian matrices, and one bad link in a unitary field, where only the
links around it leave the loop fields.

Tolerance 1e-12 relative to the largest entry: each entry adds 24 loops of at
most 6 links, some 30 products of rounding error 1e-16 each."""
import numpy as np
import pytest

import oracle
import synth
from tests import helpers as H
from tests.test_gpu_gauge_loops import cu, staples

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BETA, C1 = 2.3, -1.0 / 12.0


def links(L, kind):
    U = synth.links_haar(L, 611)
    rng = np.random.default_rng(612)
    noise = rng.standard_normal(U.shape) + 1j * rng.standard_normal(U.shape)
    if kind == "single":
        return U.astype(np.complex64).astype(np.complex128)
    if kind == "noisy":
        return U + 1e-4 * noise
    if kind == "gaussian":
        return noise
    if kind == "one":
        U[2, 5] = noise[2, 5]
    return U


@pytest.mark.parametrize("L", [(2, 2, 2, 2), (6, 2, 4, 6), (8, 4, 4, 10)])
@pytest.mark.parametrize("kind", ["unitary", "single", "noisy", "gaussian", "one"])
@pytest.mark.parametrize("scale", [1, 2])
def test_force_of_general_links_vs_oracle(L, kind, scale):
    import paper_1801_01473_amd as lq
    g = lq.Geometry(L)
    U = links(L, kind)
    U64 = lq.pack_links(g, cu(U))
    ref = oracle.gauge_force(L, U, BETA, C1)
    F = staples(lq, g, U64, BETA, C1, lq.empty_links(g).fill_(7.0), 0, scale)
    assert H.max_rel(lq.unpack_links(g, F).cpu().numpy(), ref) <= 1e-12
    staples(lq, g, U64, BETA, C1, F, 1, scale)
    assert H.max_rel(lq.unpack_links(g, F).cpu().numpy(), 2 * ref) <= 1e-12


def test_one_bad_link_leaves_the_others_alone():
    """Away from the bad link the bits are those of the unitary field."""
    import paper_1801_01473_amd as lq
    L = (8, 8, 8, 8)
    g = lq.Geometry(L)
    F = [lq.unpack_links(g, lq.gauge_force(g, lq.pack_links(g, cu(links(L, k))), BETA)).cpu().numpy()
         for k in ("unitary", "one")]
    X = (synth.site_coords(L) - synth.site_coords(L)[5] + 4) % 8 - 4
    far = np.abs(X).max(axis=1) > 3
    assert far.any() and np.array_equal(F[0][:, far], F[1][:, far])
    assert not np.array_equal(F[0][:, ~far], F[1][:, ~far])
