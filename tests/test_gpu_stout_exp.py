"""Stout smearing and its chain rule where the exponential and the workgroup
split can go wrong: half volumes below, at and past a multiple of 64, extents 2,
and smearing parameters from zero (X = 0, all eigenvalues equal) over the usual
ones (|X| < 1, no scaling) to ones that need several halvings, on near-unit and
Haar links, against the oracle (scipy's matrix exponential).

Tolerances: smearing 1e-13 while |X| < 1 (a dozen products of 1e-16 each);
each halving of X doubles the rounding error, and rho = 1.5 on Haar links takes
five (|X| up to 1.5 x 6 staples x sqrt 2 = 13 < 2^5): 32e-13.  The chain rule
carries one more factor of ten, as its products add over 18 terms."""
import numpy as np
import pytest

import oracle
import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lq():
    import paper_1801_01473_amd as lq
    return lq


def cu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


@pytest.mark.parametrize("L", [(2, 2, 2, 2), (4, 4, 4, 2), (6, 2, 4, 6), (4, 10, 2, 4)])
@pytest.mark.parametrize("rho,tol", [(0.0, 1e-13), (0.12, 1e-13), (1.5, 32e-13)])
@pytest.mark.parametrize("rough", [False, True])
def test_smearing_and_chain_rule_vs_oracle(lq, L, rho, tol, rough):
    g = lq.Geometry(L)
    U = synth.links_haar(L, 541) if rough else synth.links_exp(L, 0.2, 541)
    rng = np.random.default_rng(542)
    G = rng.standard_normal(U.shape) + 1j * rng.standard_normal(U.shape)
    chain = lq.stout_smear(g, lq.pack_links(g, cu(U)), rho, 1)
    got = lq.unpack_links(g, chain[1]).cpu().numpy()
    assert H.max_rel(got, oracle.stout_smear(L, U, rho)) <= tol
    Gp = lq.pack_links(g, cu(G))
    for mode in (0, 1):
        F = lq.unpack_links(g, lq.stout_force(g, chain, rho, Gp, mode)).cpu().numpy()
        assert H.max_rel(F, oracle.stout_force(L, U, rho, G, mode)) <= 10 * tol
