"""CG scalars inside the stencil and the update with more partials than threads.

The in-kernel sums add the partials in the order of the one-workgroup kernels, so
a run of iterations must give the same bits with either, also past 1024 partials
per system and at the most that the rule lets in.
"""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# partials (Vh / 64) and systems: 1025 and a part, 1152 x 2, 2048 (the most)
@pytest.mark.parametrize("L,n", [((2, 2, 2, 16404), 1), ((16, 16, 16, 36), 2), ((16, 16, 16, 64), 1)])
@pytest.mark.parametrize("mixed", [False, True])
def test_same_bits_as_scalar_kernels(monkeypatch, L, n, mixed):
    import paper_1801_01473_amd as lq

    monkeypatch.setenv("LQCD_DSLASH_CFG", "256,1,1,0,0,0,0,0,0,0,0,0,2,0,1")
    lq.finalize()
    g = lq.Geometry(L)
    gen = torch.Generator("cuda").manual_seed(41)
    randn = lambda s: torch.randn(s, dtype=torch.complex128, device="cuda", generator=gen)  # noqa: E731
    if mixed:  # the 12-real inner links need SU(3): diagonal phases
        ph = torch.rand((2, 4, 2, g.Vh), dtype=torch.float64, device="cuda", generator=gen)
        U = torch.zeros((2, 4, 9, g.Vh), dtype=torch.complex128, device="cuda")
        U[:, :, 0], U[:, :, 4] = torch.exp(1j * ph[:, :, 0]), torch.exp(1j * ph[:, :, 1])
        U[:, :, 8] = torch.exp(-1j * (ph[:, :, 0] + ph[:, :, 1]))
        kw = dict(inner_prec=lq.F32, inner_fmt=lq.LINKS12)
    else:
        U = 0.4 * randn((2, 4, 9, g.Vh))
        kw = {}
    b = randn((n, 3, g.Vh))
    p = lq.solver_params(mass=0.3, tol=1e-14, max_iter=40, max_refine=0, **kw)
    got = []
    for fused in ("1", "0"):
        monkeypatch.setenv("LQCD_FUSED_SCALARS", fused)
        lq.finalize()
        X, _, st = lq.cg_multishift(g, p, U, [1e-3, 0.2, 1.0], b, check=False)
        got.append((X, [s["iters"] for r in st for s in r]))
    assert got[0][1] == got[1][1] and got[0][1][0] > 10
    assert torch.isfinite(torch.view_as_real(got[0][0])).all()
    assert torch.equal(got[0][0], got[1][0])
    lq.finalize()
