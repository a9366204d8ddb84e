"""The workspace's contents on entry do not matter: a mixed multi-shift solve
that its FP64 opening phase already finishes (few, well-conditioned unknowns)
must not read the FP32 vectors, which it never wrote."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("L,mass", [((2, 2, 2, 2), 0.1), ((4, 4, 4, 2), 2.0)])
@pytest.mark.parametrize("n", [1, 2])
def test_opening_phase_that_finishes_reads_no_fp32_vectors(L, mass, n):
    import paper_1801_01473_amd as lq
    g = lq.Geometry(L)
    U = synth.links_exp(L, 0.5, 571)
    U64 = lq.pack_links(g, torch.from_numpy(np.ascontiguousarray(U)).to("cuda"))
    b_nat = synth.gaussian_even_source(L, n, 572)
    b = lq.pack_spinor(g, torch.from_numpy(b_nat).to("cuda"), 0)
    sig = [1e-3, 0.05, 1.0]
    p = lq.solver_params(mass=mass, tol=1e-10, inner_prec=lq.F32, inner_fmt=lq.LINKS12)
    lq.release_workspace()
    ws = lq._workspace(lq.solver_workspace_bytes(g, p, len(sig), n), b.device)
    out = []
    for fill in (0xFF, 0x3F):  # NaNs, finite garbage
        ws.fill_(fill)
        X, status, stats = lq.cg_multishift(g, p, U64, sig, b)
        assert status == lq.OK
        assert all(s["refine_iters"] == 0 for row in stats for s in row)
        out.append(X)
    assert torch.equal(out[0], out[1])
    Xn = lq.unpack_spinor(g, X.reshape(-1, 3, g.Vh), 0).cpu().numpy().reshape(n, 3, -1, 3)
    for j in range(n):
        for i, s in enumerate(sig):
            assert oracle.true_residual(L, U, mass, s, b_nat[j], Xn[j, i]) <= 1e-10
