"""The autotuner against the size rule's own paths (wave tiles, GEMM-1 fused with
the W-map): it never takes a fixed tile configuration where those are faster,
and its cache file keeps the decision.

Tolerance: FP64 1e-12 of the largest entry, as in test_gpu_parity."""
import numpy as np
import pytest
import torch

from oracle import contract as C
from paper_1501_05504_amd import synth

pytestmark = pytest.mark.gpu

abi = pytest.importorskip("paper_1501_05504_amd.abi")

DEV = torch.device("cuda:0")


def inputs(ml, d, mr, wl, wr):
    g = [synth.gaussian(s, 970 + i) for i, s in enumerate([(ml, wl, ml), (wl, wr, d, d), (mr, wr, mr), (ml, d, mr)])]
    return C.apply_heff(*g), [torch.tensor(x, device=DEV) for x in g]


def check(c, t, ref, calls=1):
    """W-map milliseconds of `calls` products, each compared with the oracle."""
    out = torch.empty(t[3].shape, dtype=torch.float64, device=DEV)
    c.profile_begin(calls)
    for _ in range(calls):
        out.fill_(float("nan"))
        c.apply_heff(*t, out)
        assert np.abs(out.cpu().numpy() - ref).max() < 1e-12 * np.abs(ref).max()
    return c.profile_end()[0][1]


@pytest.mark.parametrize("old_lines", [False, True], ids=["new", "with-earlier-lines"])
def test_small_products_stay_fused(tmp_path, old_lines):
    """37 x 29, d = 4, w = 6: one launch instead of three halves the time, so the
    tuned product takes it, also from the cache file, and also where that file
    has lines written before the fused kernel was among the candidates."""
    cache = tmp_path / "tune.txt"
    earlier = ["gemm:0:1:1:222:116:37:1 1", "gemm:0:1:1:148:29:174:1 1"] if old_lines else []
    cache.write_text("".join(x + "\n" for x in earlier))
    ref, t = inputs(37, 4, 29, 6, 6)
    for _ in range(2):
        c = abi.Context(0)
        try:
            c.set_autotune(True, cache)
            check(c, t, ref)
            assert check(c, t, ref, 3) == 0
        finally:
            c.close()
        lines = cache.read_text().split("\n")[:-1]
        assert lines[:len(earlier)] == earlier and len(lines) == len(earlier) + 2
        assert sum(":fused " in x for x in lines) == 1


@pytest.mark.parametrize("how", ["tile", "rule", "fused"])
def test_cached_decisions(tmp_path, how):
    """Each kind of line decides which launches run; a fused line of a shape
    that the fused kernel does not take (d = 3) runs the separate ones."""
    for (ml, d, mr), one in (((40, 4, 33), how == "fused"), ((40, 3, 33), False)):
        cache = tmp_path / ("tune%d.txt" % d)
        cache.write_text("gemm:0:1:1:%d:%d:%d:1:d%d:%s 3\n" % (6 * ml, d * mr, ml, d, how))
        ref, t = inputs(ml, d, mr, 6, 6)
        c = abi.Context(0)
        try:
            c.set_autotune(True, cache)
            assert (check(c, t, ref, 2) == 0) == one
        finally:
            c.close()
        assert len(cache.read_text().split()) == 4          # only GEMM-2 was timed


def test_capture_without_a_decision():
    """A product whose shape has not been timed is captured on the rule's path
    (no timing inside the capture) and replays with eager work in between."""
    c = abi.Context(0)
    try:
        c.set_autotune(True)
        big, tb = inputs(64, 4, 60, 6, 6)
        check(c, tb, big)                                   # sizes the workspace
        ref, t = inputs(50, 4, 40, 6, 6)
        out = torch.empty(t[3].shape, dtype=torch.float64, device=DEV)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            c.apply_heff(*t, out)
        for _ in range(3):
            out.fill_(float("nan"))
            g.replay()
            torch.cuda.synchronize()
            assert np.abs(out.cpu().numpy() - ref).max() < 1e-12 * np.abs(ref).max()
            check(c, tb, big)
    finally:
        c.close()
