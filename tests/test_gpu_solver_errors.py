"""A system whose step length overflows ends there, with the scalars inside the
stencil and the update as with kernels of their own: the solve reports it, the
rows beside it get the same bits, and the next solve is not affected.

Row 0's source has |b|^2 near the end of the double range, so |D_oe b|^2, about
twice that for a random field, is infinite at the first step."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SPLIT = "256,%d,1,0,0,0,0,0,0,0,0,0,2,0,1"


@pytest.mark.parametrize("L", [(4, 4, 4, 4), (8, 8, 8, 8)])
@pytest.mark.parametrize("n,block", [(1, 1), (3, 1), (3, 2), (4, 2)])
def test_overflowing_step_length(monkeypatch, L, n, block):
    import paper_1801_01473_amd as lq

    monkeypatch.setenv("LQCD_DSLASH_CFG", SPLIT % block)
    lq.finalize()
    g = lq.Geometry(L)
    U64 = lq.pack_links(g, torch.from_numpy(np.ascontiguousarray(synth.links_haar(L, 591))).to("cuda"))
    b = lq.pack_spinor(g, torch.from_numpy(synth.gaussian_even_source(L, n, 592)).to("cuda"), 0)
    big = b.clone()
    norm = float(torch.linalg.vector_norm(b[0]))
    big[0] *= 1.25e154 / norm  # |b|^2 = 1.56e308
    p = lq.solver_params(mass=0.1, tol=1e-8)
    sig = [1e-3, 0.05]
    out = []
    for fused in ("1", "0"):
        monkeypatch.setenv("LQCD_FUSED_SCALARS", fused)
        X, status, _ = lq.cg_multishift(g, p, U64, sig, big, check=False)
        assert status == lq.ERR_NUMERIC
        x, status, _ = lq.cg(g, p, U64, big, sigma=0.05, check=False)
        assert status == lq.ERR_NUMERIC
        out.append((X.view(torch.int64), x.view(torch.int64)))
        assert lq.cg_multishift(g, p, U64, sig, b)[1] == lq.OK
    assert torch.equal(out[0][0][1:], out[1][0][1:]) and torch.equal(out[0][1][1:], out[1][1][1:])
    lq.finalize()
