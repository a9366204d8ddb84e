"""The tuner's choice of the split stencil in the plain modes with several
right-hand sides: past the smallest lattices a plain call reads the links once for
two of them (with one a pass only when asked for, rhs_block 1), and D_oe of a solve,
which runs on one link field, is tuned apart from it, under a key of its own."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("L,apart", [((8, 8, 8, 8), False), ((16, 16, 16, 8), False),
                                     ((16, 16, 16, 16), True)])
@pytest.mark.parametrize("prec", [0, 1])
def test_plain_calls_and_solves(monkeypatch, tmp_path, L, apart, prec):
    import paper_1801_01473_amd as lq

    monkeypatch.delenv("LQCD_DSLASH_CFG", raising=False)
    monkeypatch.setenv("LQCD_RHS_PAIRS", "0")
    path = tmp_path / "cache.txt"
    monkeypatch.setenv("LQCD_TUNE_CACHE", str(path))
    lq.finalize()
    g = lq.Geometry(L)
    U64 = torch.zeros((2, 4, 9, g.Vh), dtype=torch.complex128, device="cuda")
    U64[:, :, 0] = U64[:, :, 4] = U64[:, :, 8] = 1.0
    U = lq.convert_links(g, U64, lq.F64, lq.LINKS18, lq.F32, lq.LINKS12) if prec else U64
    gen = torch.Generator("cuda").manual_seed(52)
    b = torch.randn((3, 3, g.Vh), dtype=torch.complex128, device="cuda", generator=gen)

    def lines():
        return [(k, [int(v) for v in cfg.split(",")])
                for k, cfg in (x.split(";") for x in path.read_text().splitlines())]

    for n in (1, 2, 3):
        lq.apply_A(g, U, 0.1, 0.2, b[:n].to(U.dtype).contiguous())
    plain = lines()
    assert len(plain) == 6
    for key, cfg in plain:
        n = int(key.split("/n")[1].split("/")[0])
        assert cfg[-1] == 0 or not apart or cfg[1] == min(n, 2), (key, cfg)
    kw = dict(inner_prec=lq.F32, inner_fmt=lq.LINKS12, mixed_switch=0.0) if prec else {}
    lq.cg_multishift(g, lq.solver_params(mass=1.0, tol=1e-6, max_refine=0, **kw), U64, [0.1, 1.0], b[:2].contiguous(), check=False)
    new = [k for k, _ in lines()[6:] if f"/p{prec}/f{1 if prec else 0}/n2/b0/m0" in k]
    assert new == ([k + "/solve" for k, _ in plain if f"/p{prec}/f{1 if prec else 0}/n2/b0/m0" in k]
                   if apart else [])
    lq.finalize()
