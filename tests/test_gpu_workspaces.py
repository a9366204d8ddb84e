"""Calls that return before their kernels have run keep their workspace to
themselves: gauge forces on two streams, and in a captured graph whose replays
alternate with eager calls, give the bits of calls made one after the other."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def case():
    import paper_1801_01473_amd as lq
    L = (16, 16, 16, 16)
    g = lq.Geometry(L)
    U = [lq.pack_links(g, torch.from_numpy(np.ascontiguousarray(synth.links_exp(L, 0.5, s))).to("cuda"))
         for s in (601, 602)]
    ref = [lq.gauge_force(g, u, 2.3) for u in U]
    torch.cuda.synchronize()
    return lq, g, U, ref


def test_two_streams(case):
    lq, g, U, ref = case
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    F = [[lq.empty_links(g) for _ in range(8)] for _ in U]
    torch.cuda.synchronize()
    for i in range(8):
        for k, s in enumerate(streams):
            with torch.cuda.stream(s):
                lq.gauge_force(g, U[k], 2.3, out=F[k][i])
    torch.cuda.synchronize()
    for k in range(2):
        assert all(torch.equal(f, ref[k]) for f in F[k])


def test_captured(case):
    lq, g, U, ref = case
    F = lq.empty_links(g)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        lq.gauge_force(g, U[0], 2.3, out=F)
    lq.release_workspace()
    for _ in range(4):
        F.zero_()
        other = lq.gauge_force(g, U[1], 2.3)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(F, ref[0]) and torch.equal(other, ref[1])


@pytest.mark.parametrize("keep", [0, 1 << 40])
def test_force_where_twice_the_workspace_does_not_fit(case, monkeypatch, keep):
    """Without the memory for twice the required workspace the force is formed
    in two passes of three planes, and the required workspace is all that is kept."""
    lq, g, U, ref = case
    monkeypatch.setattr(lq, "_KEEP_TWICE", keep)
    need = int(lq._fn("lqcd_gauge_force_staples_workspace_bytes")(g.c()))
    F = lq.empty_links(g)
    lq.release_workspace()
    empty = torch.empty

    def limited(*a, **k):
        if a[0] == 2 * need:
            raise torch.OutOfMemoryError("limit")
        return empty(*a, **k)

    monkeypatch.setattr(torch, "empty", limited)
    lq.gauge_force(g, U[0], 2.3, out=F)
    torch.cuda.synchronize()
    assert [w.numel() for w in lq._workspaces().values()] == [need]
    assert float((F - ref[0]).abs().max()) <= 1e-13 * float(ref[0].abs().max())
