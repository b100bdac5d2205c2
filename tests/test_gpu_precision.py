"""Errors of fp32 gradients against the fp64 oracle, compared between the two
engines of the library: the fused one must not be less exact than the generic
one (CAVS_GENERIC=1), which sums the forget blocks of the slots before dX's
product, forms every product on the fp32 instruction and splits its long
contractions into chains of its own.  Relative 2-norm errors; rounding makes
either one differ by a few per cent from seed to seed, so 5 % are allowed."""
import numpy as np
import pytest

from parity import oracle_sharded
from paper_1712_04048_amd import binding as B
from paper_1712_04048_amd import workloads as W
from paper_1712_04048_amd.runner import Batch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = B.Context(0)
    yield c
    c.close()


def _errors(wl, ctx, monkeypatch, keys):
    want = oracle_sharded(wl)
    out = {}
    for mode in ("0", "1"):
        monkeypatch.setenv("CAVS_GENERIC", mode)
        got = Batch(wl, ctx).run()
        out[mode] = {k: float(np.linalg.norm(got[k] - want[k]) / np.linalg.norm(want[k]))
                     for k in keys}
    print("errors fused / generic: %s" % {k: "%.3g / %.3g" % (out["0"][k], out["1"][k])
                                          for k in keys}, flush=True)
    return out["0"], out["1"]


@pytest.mark.parametrize("H,N,K", [(320, 2, 30), (256, 3, 60), (128, 4, 60)])
def test_dx_with_several_slots(ctx, monkeypatch, H, N, K):
    """Inputs at every vertex: dX contracts 3 + N blocks of dA."""
    rng = np.random.Generator(np.random.PCG64(H))
    make = (lambda n: W.random_split_tree(n, rng)) if N == 2 else (lambda n: W.nary_tree(n, N, rng))
    wl = W.make_workload("dx", [make(int(n)) for n in rng.integers(3, 30, size=K)], N=N, D=100,
                         H=H, C=5, sigma=0.05, rng=rng, inputs="all", labels="all")
    fused, generic = _errors(wl, ctx, monkeypatch, ["dX"])
    assert fused["dX"] <= 1.05 * generic["dX"]


def test_du_of_long_contractions(ctx, monkeypatch):
    """Some 4 700 internal vertices at H = 512: the longest chains of the
    split lazy products."""
    fused, generic = _errors(W.config_treelstm_sst(0), ctx, monkeypatch, ["dU", "dWx"])
    for k in fused:
        assert fused[k] <= 1.05 * generic[k], k
