"""Mixed CG of well-conditioned systems, whose FP32 residual falls so far between
two looks of the host that the FP64 one is up to a few times larger: the solve must
restart its directions and converge like one that looks more often, at every
distance between looks.  (Directions kept at a ratio of 3.7 diverged.)"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("L,mass,sigma", [((6, 4, 4, 6), 0.1, 0.05), ((8, 8, 8, 8), 0.1, 0.05),
                                          ((4, 4, 4, 4), 0.3, 0.0), ((6, 4, 4, 6), 0.05, 0.02)])
@pytest.mark.parametrize("n", [1, 2, 4])
def test_every_poll_interval_converges(L, mass, sigma, n):
    import paper_1801_01473_amd as lq
    g = lq.Geometry(L)
    U = synth.links_exp(L, 0.5, 563)
    U64 = lq.pack_links(g, torch.from_numpy(np.ascontiguousarray(U)).to("cuda"))
    b_nat = synth.gaussian_even_source(L, n, 564)
    b = lq.pack_spinor(g, torch.from_numpy(b_nat).to("cuda"), 0)
    iters = []
    for poll in (10, 0, 24, 28, 31, 35, 40, 47, 55, 62):
        p = lq.solver_params(mass=mass, tol=1e-10, inner_prec=lq.F32, inner_fmt=lq.LINKS12,
                             poll_interval=poll)
        x, status, st = lq.cg(g, p, U64, b, sigma=sigma, check=False)
        assert status == lq.OK, (poll, st)
        iters.append(max(s["iters"] + s["refine_iters"] for s in st))
        xn = lq.unpack_spinor(g, x, 0).cpu().numpy()
        for j in range(n):
            assert oracle.true_residual(L, U, mass, sigma, b_nat[j], xn[j]) <= 1e-10
    # an FP32 residual that has stopped falling costs at most one look's iterations
    # each time, and a solve has few of them
    assert max(iters) <= 2 * iters[0] + 62, iters
