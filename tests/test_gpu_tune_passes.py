"""The tuner's choice of the split stencil in the plain modes: with several
right-hand sides it reads the links once for two of them, with one a pass only
when asked for (rhs_block 1)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("L", [(4, 4, 4, 4), (8, 8, 8, 8), (12, 12, 12, 12)])
@pytest.mark.parametrize("prec", [0, 1])
def test_split_stencil_reads_links_once_for_two(monkeypatch, tmp_path, L, prec):
    import paper_1801_01473_amd as lq

    monkeypatch.delenv("LQCD_DSLASH_CFG", raising=False)
    path = tmp_path / "cache.txt"
    monkeypatch.setenv("LQCD_TUNE_CACHE", str(path))
    lq.finalize()
    g = lq.Geometry(L)
    U = lq.pack_links(g, torch.from_numpy(np.ascontiguousarray(synth.links_haar(L, 631))).to("cuda"), prec, 0)
    for n in (1, 2, 3):
        x = lq.pack_spinor(g, torch.from_numpy(synth.gaussian_field(L, n, 632)).to("cuda"), 0, prec)
        lq.apply_A(g, U, 0.1, 0.2, x)
    lines = [x.split(";") for x in path.read_text().splitlines()]
    assert len(lines) >= 6
    for key, cfg in lines:
        cfg = [int(v) for v in cfg.split(",")]
        n = int(key.split("/n")[1].split("/")[0])
        assert cfg[-1] == 0 or cfg[1] == min(n, 2), (key, cfg)
    lq.finalize()
