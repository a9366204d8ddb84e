"""Packing and unpacking at the edges of their 256-thread workgroups.

Every value is moved, not computed with, so the comparisons are exact; the guard
words behind each output must keep their value.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def site_order(L):
    """[parity][Vh] lexicographic site numbers (x fastest) in half-index order."""
    x, y, z, t = L
    lex = np.arange(x * y * z * t)
    par = (lex % x + lex // x % y + lex // (x * y) % z + lex // (x * y * z)) % 2
    return np.stack([lex[par == p] for p in (0, 1)])


def guarded(shape, dtype):
    n = int(np.prod(shape))
    flat = torch.full((n + 64,), 7.5, dtype=dtype, device="cuda")
    return flat, flat[:n].view(shape)


# 4 V = 64 (a quarter workgroup), 384 (one and a half), 512 (exact), 1152
@pytest.mark.parametrize("L", [(2, 2, 2, 2), (4, 2, 2, 6), (4, 4, 4, 2), (6, 2, 6, 4)])
@pytest.mark.parametrize("n", [1, 3])
def test_pack_and_unpack_are_exact(L, n):
    import paper_1801_01473_amd as lq

    g = lq.Geometry(L)
    rng = np.random.default_rng(5)
    cplx = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)  # noqa: E731
    order = site_order(L)

    nat = cplx(4, g.V, 3, 3)
    flat, U = guarded((2, 4, 9, g.Vh), torch.complex128)
    lq.pack_links(g, torch.from_numpy(nat).cuda(), out=U)
    want = nat[:, order].transpose(1, 0, 3, 4, 2).reshape(2, 4, 9, g.Vh)
    assert np.array_equal(U.cpu().numpy(), want)
    assert (flat[-64:] == 7.5).all()
    flat, back = guarded((4, g.V, 3, 3), torch.complex128)
    lq.unpack_links(g, U, out=back)
    assert np.array_equal(back.cpu().numpy(), nat)
    assert (flat[-64:] == 7.5).all()

    for prec, dt in ((lq.F64, torch.complex128), (lq.F32, torch.complex64)):
        for par in (0, 1):
            v = torch.from_numpy(cplx(n, 3, g.Vh)).cuda().to(dt)
            flat, out = guarded((n, g.V, 3), torch.complex128)
            lq.unpack_spinor(g, v, par, out=out)
            want = np.zeros((n, g.V, 3), complex)
            want[:, order[par]] = v.cpu().numpy().astype(complex).transpose(0, 2, 1)
            assert np.array_equal(out.cpu().numpy(), want)
            assert (flat[-64:] == 7.5).all()
            assert torch.equal(lq.pack_spinor(g, out, par, prec), v)
