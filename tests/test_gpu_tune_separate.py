"""The tuner's choice of the CG update for solves whose scalars stay in kernels of
their own: the split stencil gets no credit there for launches that it does not
save, so a kept choice of it, made with that credit, is not taken over, while a
kept choice of another kernel is."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("how", ["one_shift_per_window", "switched_off"])
def test_lines_tuned_with_the_credit(monkeypatch, tmp_path, how):
    import paper_1801_01473_amd as lq

    monkeypatch.delenv("LQCD_DSLASH_CFG", raising=False)
    path = tmp_path / "cache.txt"
    monkeypatch.setenv("LQCD_TUNE_CACHE", str(path))
    L = (8, 4, 4, 4)
    g = lq.Geometry(L)
    U64 = lq.pack_links(g, torch.from_numpy(np.ascontiguousarray(synth.links_exp(L, 0.5, 621))).to("cuda"))
    b = lq.pack_spinor(g, torch.from_numpy(synth.gaussian_even_source(L, 1, 622)).to("cuda"), 0)

    def keys(**kw):
        """The CG updates' lines after a solve that starts from the file."""
        lq.finalize()
        lq.cg_multishift(g, lq.solver_params(mass=0.5, tol=1e-8, **kw), U64, [0.0, 0.1], b)
        return [x.split(";") for x in path.read_text().splitlines() if "/m2" in x]

    def separate():
        if how == "switched_off":
            monkeypatch.setenv("LQCD_FUSED_SCALARS", "0")
            got = keys()
            monkeypatch.delenv("LQCD_FUSED_SCALARS")
            return got
        return keys(shift_window=1)

    (key, _), = keys()
    assert keys() == keys() and len(keys()) == 1  # found again
    other = "64,1,0,0,0,0,0,0,0,0,0,0,2,0"
    split = "256,1,1,0,0,0,0,0,0,0,0,0,2,1"
    path.write_text(f"{key};{other}\n")
    assert separate() == [[key, other]]
    path.write_text(f"{key};{split}\n")
    assert keys() == [[key, split]]
    got = separate()
    assert got[0] == [key, split] and [k for k, _ in got[1:]] == [key + "/sep"]
    assert separate() == got  # and that one is found again
    lq.finalize()
