"""A NaN stays in its own graph.  The input row of position 0's vertex (the
leaf with the smallest id) is NaN; every state and input gradient of the other
graphs is bit for bit what it is without the NaN, at every engine path a vertex
with absent child slots takes: split-K, tiles, the level loop (forced on and
off), two to four slots, trees and graphs, both precisions.  The one exception:
in a batch large enough for the split pull product, the 128 rows that share a
tile with the NaN are formed on the fp32 instruction, so their sums round in
another order: there 2e-6 of the largest value, some 30 fp32 roundings."""
import numpy as np
import pytest

from paper_1712_04048_amd import binding as B
from paper_1712_04048_amd import workloads as W
from paper_1712_04048_amd.runner import Batch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = B.Context(0)
    yield c
    c.close()


def _graphs(kind, N, K, rng):
    if kind == "unary":   # one child where two are possible, at several depths
        return [[[-1, -1], [0, -1], [-1, -1], [2, -1], [1, 3], [4, -1]]] * K
    if kind == "dag":
        return [W.random_dag(int(n), N, rng) for n in rng.integers(4, 12, size=K)]
    return [W.nary_tree(int(n), N, rng) for n in rng.integers(3, 12, size=K)]


# (H, N, kind, K, bf16)
CASES = [(64, 3, "nary", 20, False), (192, 4, "nary", 12, False), (512, 3, "nary", 9, False),
         (256, 4, "nary", 90, False), (128, 3, "nary", 1500, False), (320, 2, "unary", 10, False),
         (512, 2, "unary", 40, False), (768, 2, "unary", 5, False), (128, 2, "dag", 20, False),
         (256, 4, "dag", 30, False), (320, 2, "unary", 10, True), (1024, 2, "unary", 6, True),
         (1024, 2, "unary", 100, True), (512, 2, "unary", 1200, True)]


@pytest.mark.parametrize("loop", ["0", "1"])
@pytest.mark.parametrize("H,N,kind,K,bf16", CASES)
def test_nan_in_position_zero(ctx, monkeypatch, H, N, kind, K, bf16, loop):
    monkeypatch.setenv("CAVS_XCD_LOOP", loop)
    rng = np.random.Generator(np.random.PCG64(H + N + K))
    wl = W.make_workload("nan", _graphs(kind, N, K, rng), N=N, D=12, H=H, C=5, sigma=0.1,
                         prec=W.PREC_BF16 if bf16 else W.PREC_FP32, rng=rng, inputs="all",
                         labels="all", dag=kind == "dag")
    print("nan H=%d N=%d %s K=%d V=%d loop=%s" % (H, N, kind, K, wl.V, loop), flush=True)
    clean = Batch(wl, ctx).run()
    assert (wl.child[0] < 0).all() and wl.pull_idx[0] >= 0
    wl.X[wl.pull_idx[0]] = np.nan
    got = Batch(wl, ctx).run()
    others = np.arange(wl.tree_offsets[1], wl.V)
    assert np.isnan(got["h"][0]).all()
    split_pull = not bf16 and -(-wl.n_x // 128) * (4 * H // 128) >= 256
    rows = wl.pull_idx[others]
    for k, at in (("h", others), ("c", others), ("dX", rows)):
        a, b = got[k][at], clean[k][at]
        assert np.isfinite(a).all(), k
        if split_pull:
            assert np.abs(a - b).max() <= 2e-6 * np.abs(b).max(), k
        else:
            assert np.array_equal(a, b), k
