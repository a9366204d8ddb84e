"""A right-hand side of zeros in a batch: its system is finished before the first
iteration, and the others must not notice, whatever the workspace held on entry.

With the scalars inside the stencil and the update (pinned split stencil) the
finished system shares its launches with the live ones, alone in its group of
right-hand sides or beside a live one, as the first, a middle and the last row,
in pairs and in separate rows.  Its solution is zero, and the others are the same
bits as with the scalars in kernels of their own."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SPLIT = "256,%d,1,0,0,0,0,0,0,0,0,0,2,0,1"
SIG = [1e-3, 0.05, 1.0]


@pytest.mark.parametrize("L", [(2, 2, 2, 2), (8, 4, 4, 4)])
@pytest.mark.parametrize("n,zero", [(2, (0,)), (2, (1,)), (4, (0, 1)), (5, (0, 2, 4))])
@pytest.mark.parametrize("block", [1, 2])
@pytest.mark.parametrize("mixed", [False, True])
def test_zero_rows_beside_others(monkeypatch, L, n, zero, block, mixed):
    import paper_1801_01473_amd as lq

    monkeypatch.setenv("LQCD_DSLASH_CFG", SPLIT % block)
    lq.finalize()
    g = lq.Geometry(L)
    U = synth.links_exp(L, 0.5, 581)
    U64 = lq.pack_links(g, torch.from_numpy(np.ascontiguousarray(U)).to("cuda"))
    b_nat = synth.gaussian_even_source(L, n, 582)
    b_nat[list(zero)] = 0
    b = lq.pack_spinor(g, torch.from_numpy(b_nat).to("cuda"), 0)
    kw = dict(inner_prec=lq.F32, inner_fmt=lq.LINKS12) if mixed else {}
    p = lq.solver_params(mass=0.1, tol=1e-10, **kw)
    lq.release_workspace()
    ws = lq._workspace(lq.solver_workspace_bytes(g, p, len(SIG), n), b.device)
    ref = None
    for fused, fill in (("0", 0), ("1", 0), ("1", 0x80), ("1", 0xC3), ("1", 0x7F), ("1", 0xFF)):
        monkeypatch.setenv("LQCD_FUSED_SCALARS", fused)
        ws.fill_(fill)
        X, status, st = lq.cg_multishift(g, p, U64, SIG, b)
        assert status == lq.OK
        ref = X if ref is None else ref
        assert torch.equal(X, ref), (fused, fill)
        for j in range(n):
            assert (st[j][0]["iters"] == 0) == (j in zero)
            assert (X[j].abs().max().item() == 0.0) == (j in zero)
    Xn = lq.unpack_spinor(g, ref.reshape(-1, 3, g.Vh), 0).cpu().numpy().reshape(n, 3, -1, 3)
    for j in set(range(n)) - set(zero):
        for i, s in enumerate(SIG):
            assert oracle.true_residual(L, U, 0.1, s, b_nat[j], Xn[j, i]) <= 1e-10
    lq.finalize()
