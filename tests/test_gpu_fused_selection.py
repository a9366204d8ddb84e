"""Which solves compute their scalars inside the stencil and the update.

The tests that compare that path with kernels of its own agree bit for bit also
if both sides run the same kernels, so here the selection itself is read back:
with the split stencil pinned, every shape of those tests takes the path, as
separate rows and in pairs, and none does when it is switched off or where a
solve has several shifts and one iteration a window."""
import re

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SPLIT = "256,%d,1,0,0,0,0,0,0,0,0,0,2,0,1"
LINE = re.compile(r"phase (f32|f64) n=(\d+) pairs=(\d): D_oe sp=(\d), D_eo sp=(\d) B=(\d), fused=(\d)")


def phases(lq, capfd, L, n, mixed, single=False, **kw):
    """(precision, pairs, split, block, fused) of each phase of a short solve."""
    g = lq.Geometry(L)
    U = torch.zeros((2, 4, 9, g.Vh), dtype=torch.complex128, device="cuda")
    U[:, :, 0] = U[:, :, 4] = U[:, :, 8] = 1.0
    gen = torch.Generator("cuda").manual_seed(51)
    b = torch.randn((n, 3, g.Vh), dtype=torch.complex128, device="cuda", generator=gen)
    if mixed:
        kw.update(inner_prec=lq.F32, inner_fmt=lq.LINKS12)
    p = lq.solver_params(mass=1.0, tol=1e-6, max_refine=0, **kw)
    capfd.readouterr()
    if single:
        lq.cg(g, p, U, b, check=False)
    else:
        lq.cg_multishift(g, p, U, [0.1, 1.0], b, check=False)
    return [(m[0], int(m[2]), int(m[4]), int(m[5]), int(m[6]))
            for m in LINE.findall(capfd.readouterr().err)]


@pytest.fixture
def lq(monkeypatch):
    import paper_1801_01473_amd as lq
    monkeypatch.setenv("LQCD_DEBUG", "1")
    monkeypatch.delenv("LQCD_FUSED_SCALARS", raising=False)
    lq.finalize()
    yield lq
    lq.finalize()


@pytest.mark.parametrize("L,n,block", [((2, 2, 2, 2), 1, 1), ((2, 2, 2, 2), 2, 2), ((8, 8, 8, 8), 3, 2),
                                       ((8, 8, 8, 8), 4, 1), ((2, 2, 2, 16404), 1, 1),
                                       ((16, 16, 16, 64), 1, 1)])
@pytest.mark.parametrize("mixed", [False, True])
def test_fused_where_the_comparisons_assume_it(lq, monkeypatch, capfd, L, n, block, mixed):
    monkeypatch.setenv("LQCD_DSLASH_CFG", SPLIT % block)
    pairs = 1 if mixed and n % 2 == 0 else 0
    want = [("f64", 0, 1, block, 1)] + ([("f32", pairs, 1, 2 if pairs else block, 1)] if mixed else [])
    assert phases(lq, capfd, L, n, mixed) == want
    assert phases(lq, capfd, L, n, mixed, single=True) == [("f32" if mixed else "f64", 0, 1, block, 1)]
    assert all(ph[-1] == 0 for ph in phases(lq, capfd, L, n, mixed, shift_window=1))
    monkeypatch.setenv("LQCD_FUSED_SCALARS", "0")
    assert all(ph[-1] == 0 for ph in phases(lq, capfd, L, n, mixed))
    assert all(ph[-1] == 0 for ph in phases(lq, capfd, L, n, mixed, single=True))


@pytest.mark.parametrize("L,n,fused", [((8, 8, 8, 16), 2, 1), ((8, 8, 8, 16), 8, 1),
                                       ((16, 16, 16, 16), 2, 0), ((12, 12, 12, 24), 8, 0)])
def test_pairs_fuse_up_to_fewer_partials(lq, monkeypatch, capfd, L, n, fused):
    """nb^2 n partials of 2^13, 2^15 and 2^19, 2^20; as separate rows up to 2^20."""
    monkeypatch.setenv("LQCD_DSLASH_CFG", SPLIT % 2)
    assert phases(lq, capfd, L, n, True)[1] == ("f32", 1, 1, 2, fused)
    monkeypatch.setenv("LQCD_RHS_PAIRS", "0")
    assert phases(lq, capfd, L, n, True)[1] == ("f32", 0, 1, 2, 1)
