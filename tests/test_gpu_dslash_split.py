"""The direction-split stencil and the scalars computed inside the CG kernels.

The split kernel adds the eight hops in the order of the one-thread-per-site
kernel, so with either pinned D_oe, D_eo and the operator must agree bit for
bit, in every precision and link format, for RHS counts that leave a block
short, at half volumes below, at and past a multiple of 64.  Solves with it
(single system, several, mixed multi-shift with and without right-hand-side
pairs, graphs on and off, with the scalars inside the stencil and the update or
in kernels of their own) must reach the true residual, judged by the oracle, and
agree bit for bit."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LATS = [(2, 2, 2, 2), (4, 2, 6, 4), (4, 4, 4, 2), (6, 4, 4, 6), (8, 4, 4, 4)]
PLAIN = "256,%d,1,0,0,0,0,0,0,0,0,0,2,0,0"
SPLIT = "256,%d,%d,0,0,0,0,0,0,0,0,0,2,0,1"


@pytest.fixture(scope="module")
def lq():
    import paper_1801_01473_amd as lq
    return lq


def cu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


@pytest.mark.parametrize("L", LATS)
@pytest.mark.parametrize("anti", [True, False])
@pytest.mark.parametrize("fmt", [0, 1, 2, 3])
@pytest.mark.parametrize("prec", [0, 1])
def test_same_bits_as_one_thread_per_site(lq, monkeypatch, L, anti, fmt, prec):
    g = lq.Geometry(L, anti)
    U = lq.pack_links(g, cu(synth.links_haar(L, 561)), prec, fmt)
    for n in (1, 2, 3):
        x = [lq.pack_spinor(g, cu(synth.gaussian_field(L, n, 562)), p, prec) for p in (0, 1)]
        ref = None
        for cfg in (PLAIN % 1, SPLIT % (1, 0), SPLIT % (1, 1), SPLIT % (2, 1)):
            if cfg.startswith("256,2") and n < 2:
                continue
            monkeypatch.setenv("LQCD_DSLASH_CFG", cfg)
            got = (lq.doe(g, U, x[0]), lq.deo(g, U, x[1]), lq.apply_A(g, U, 0.1, 0.2, x[0]))
            if ref is None:
                ref = got
            for a, b in zip(got, ref):
                assert torch.equal(a, b), (cfg, n)


def residuals(lq, g, L, U, mass, sig, b_nat, X):
    Xn = lq.unpack_spinor(g, X.reshape(-1, 3, g.Vh), 0).cpu().numpy().reshape(
        len(b_nat), len(sig), -1, 3)
    return max(oracle.true_residual(L, U, mass, s, b_nat[j], Xn[j, i])
               for j in range(len(b_nat)) for i, s in enumerate(sig))


@pytest.mark.parametrize("L", [(2, 2, 2, 2), (4, 4, 4, 2), (6, 4, 4, 6), (8, 8, 8, 8)])
@pytest.mark.parametrize("n,block", [(1, 1), (2, 1), (3, 2), (4, 2)])
@pytest.mark.parametrize("prec", [0, 1])
def test_solves_with_fused_scalars(lq, monkeypatch, L, n, block, prec):
    monkeypatch.setenv("LQCD_DSLASH_CFG", SPLIT % (block, 1))
    lq.finalize()
    g = lq.Geometry(L)
    U = synth.links_exp(L, 0.5, 563)
    U64 = lq.pack_links(g, cu(U))
    b_nat = synth.gaussian_even_source(L, n, 564)
    b = lq.pack_spinor(g, cu(b_nat), 0)
    sig = [1e-3, 0.05, 1.0]
    kw = dict(mass=0.1, tol=1e-10)
    if prec:
        kw.update(inner_prec=lq.F32, inner_fmt=lq.LINKS12)
    out = []
    for graph in (1, 0):
        p = lq.solver_params(use_graph=graph, **kw)
        X, _, st = lq.cg_multishift(g, p, U64, sig, b)
        assert residuals(lq, g, L, U, 0.1, sig, b_nat, X) <= 1e-10
        # (mixed: the FP64 residual is recomputed at these polls)
        x, _, _ = lq.cg(g, lq.solver_params(use_graph=graph, poll_interval=10, **kw), U64, b,
                        sigma=0.05)
        assert residuals(lq, g, L, U, 0.1, [0.05], b_nat, x) <= 1e-10
        out.append((X, x))
        if graph:
            # the scalars in kernels of their own: the same bits
            monkeypatch.setenv("LQCD_FUSED_SCALARS", "0")
        else:
            monkeypatch.delenv("LQCD_FUSED_SCALARS")
            X, _, st = lq.cg_multishift(g, p, U64, sig, b)
            out.append((X, x))
    for X, x in out[1:]:
        assert torch.equal(out[0][0], X) and torch.equal(out[0][1], x)
    if prec and n % 2 == 0:  # pairs: the same bits as separate rows
        monkeypatch.setenv("LQCD_RHS_PAIRS", "0")
        monkeypatch.setenv("LQCD_DSLASH_CFG", SPLIT % (2, 1))
        X0 = lq.cg_multishift(g, p, U64, sig, b)[0]
        monkeypatch.delenv("LQCD_RHS_PAIRS")
        X1 = lq.cg_multishift(g, p, U64, sig, b)[0]
        assert torch.equal(X0, X1)
    lq.finalize()


@pytest.mark.parametrize("n", [1, 2])
def test_fused_scalars_stop_on_the_iteration_limit_and_on_nan(lq, monkeypatch, n):
    """max_iter stops every system at that count; a NaN source is reported and
    leaves the other calls alone."""
    monkeypatch.setenv("LQCD_DSLASH_CFG", SPLIT % (1, 1))
    lq.finalize()
    L = (4, 4, 4, 4)
    g = lq.Geometry(L)
    U64 = lq.pack_links(g, cu(synth.links_haar(L, 565)))
    b = lq.pack_spinor(g, cu(synth.gaussian_even_source(L, n, 566)), 0)
    p = lq.solver_params(mass=0.02, tol=1e-12, max_iter=7, max_refine=0)
    _, status, st = lq.cg(g, p, U64, b, check=False)
    assert status == lq.ERR_NOT_CONVERGED and all(s["iters"] == 7 for s in st)
    bad = b.clone()
    bad[0, 0, 0] = float("nan")
    p = lq.solver_params(mass=0.02)
    assert lq.cg(g, p, U64, bad, check=False)[1] == lq.ERR_NUMERIC
    assert lq.cg(g, p, U64, b, check=False)[1] == lq.OK
    lq.finalize()
