"""The exponential of the link update over the range of its scaling.

exp(X), |X| = |eps H|: each of the log2 |X| squarings doubles a relative error of
about 20 roundings, and reunitarization, the products and the reference add a
few dozen: 2e-14 max(1, |X|) holds with room.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# |H| is about 3: no scaling, its edge, one squaring, several; half volumes 8
# (part of a workgroup), 72
@pytest.mark.parametrize("eps", [0.0, 1e-6, 0.05, 0.33, 0.5, -4.0])
@pytest.mark.parametrize("L", [(2, 2, 2, 2), (6, 2, 6, 2)])
def test_link_update_exponential(eps, L):
    import paper_1801_01473_amd as lq

    g = lq.Geometry(L)
    rng = np.random.default_rng(17)
    h = rng.standard_normal((4, g.V, 3, 3)) + 1j * rng.standard_normal((4, g.V, 3, 3))
    h = 0.5 * (h + h.conj().swapaxes(-1, -2))
    h -= np.trace(h, axis1=-2, axis2=-1)[..., None, None] / 3 * np.eye(3)
    h[0, 0] = 0.0  # exp(0)
    h[1, 0] = np.diag([1.0, 1.0, -2.0])  # two equal eigenvalues
    U = synth.links_haar(L, 77).reshape(4, g.V, 3, 3)
    w, v = np.linalg.eigh(h)
    want = np.einsum("...ab,...b,...cb,...cd->...ad", v, np.exp(1j * eps * w), v.conj(), U)
    cu = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")  # noqa: E731
    U64 = lq.pack_links(g, cu(U))
    lq.md_update_links(g, U64, lq.pack_links(g, cu(h)), eps)
    got = lq.unpack_links(g, U64).cpu().numpy()
    norm = abs(eps) * np.sqrt((abs(h) ** 2).sum((-1, -2)))
    err = abs(got - want).max((-1, -2))
    assert (err <= 2e-14 * np.maximum(1.0, norm)).all(), (err / np.maximum(1.0, norm)).max()
