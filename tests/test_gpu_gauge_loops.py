"""The gauge force through loop fields at the edges of its wave and workspace
splits: half volumes below, at and past a multiple of 64, extents 2 (loops
that wrap onto themselves), both workspace sizes (the required one, in which
three planes at a time add up, and twice that, one pass over all six), against
the oracle's loop enumeration.

Tolerance 1e-12 relative to the largest entry: each entry adds 24 loops of at
most 6 links, some 30 products of rounding error 1e-16 each."""
import ctypes

import numpy as np
import pytest

import oracle
import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lq():
    import paper_1801_01473_amd as lq
    return lq


def cu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def staples(lq, g, U64, beta, c1, F, accumulate, scale):
    fn = lq._fn("lqcd_gauge_force_staples")
    n = int(lq._fn("lqcd_gauge_force_staples_workspace_bytes")(g.c()))
    guarded = torch.full((int(scale * n) + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    ws = guarded[:int(scale * n)]
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    st = fn(g.c(), ptr(U64), beta, c1, accumulate, ptr(F), ptr(ws), ws.numel(),
            ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == lq.OK, lq.last_error()
    assert bool((guarded[int(scale * n):] == 0x5A).all()), "write past the workspace"
    return F


@pytest.mark.parametrize("L", [(2, 2, 2, 2), (2, 4, 2, 6), (4, 4, 4, 2), (6, 2, 4, 6),
                               (10, 6, 4, 2), (8, 4, 4, 10)])
@pytest.mark.parametrize("c1", [-1.0 / 12.0, 0.0])
@pytest.mark.parametrize("scale", [1, 1.99, 2])
def test_loop_field_force_vs_oracle(lq, L, c1, scale):
    g = lq.Geometry(L)
    U = synth.links_haar(L, 531)
    U64 = lq.pack_links(g, cu(U))
    ref = oracle.gauge_force(L, U, 2.3, c1)
    F = staples(lq, g, U64, 2.3, c1, lq.empty_links(g).fill_(7.0), 0, scale)
    got = lq.unpack_links(g, F).cpu().numpy()
    assert H.max_rel(got, ref) <= 1e-12
    staples(lq, g, U64, 2.3, c1, F, 1, scale)
    assert H.max_rel(lq.unpack_links(g, F).cpu().numpy(), 2 * ref) <= 1e-12
