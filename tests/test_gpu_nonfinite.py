"""Infinities and values near the largest float as operands of the split
products.  They have no bf16 parts; the states and gradients are those of the
fp32 instruction all the same: an infinite input saturates its gates, whatever
the size of the batch, and a product that a small batch forms on the fp32
instruction and a large one on split operands gives both the same.  The oracle
evaluates the same batches in fp64 (1e-4 of each tensor's largest value, the
fp32 bar of the parity tests)."""
import numpy as np
import pytest

from parity import check, oracle_sharded
from paper_1712_04048_amd import binding as B
from paper_1712_04048_amd import workloads as W
from paper_1712_04048_amd.runner import Batch

pytestmark = pytest.mark.gpu

HUGE = np.float32(3.3999e38)     # finite, above bf16's largest value


@pytest.fixture(scope="module")
def ctx():
    c = B.Context(0)
    yield c
    c.close()


def _trees(K, inputs, rng, H=512, D=20, N=2):
    graphs = [W.complete_tree(2)] * K if N == 2 else [W.chain(3)] * K
    return W.make_workload("nonfinite", graphs, N=N, D=D, H=H, C=5, sigma=0.05, rng=rng,
                           inputs=inputs, labels="all")


@pytest.mark.parametrize("K", [40, 1200])     # below and above the line of the split pull product
@pytest.mark.parametrize("inputs", ["leaves", "all"])
def test_large_inputs(ctx, K, inputs):
    """Every gradient too: a saturated gate's dA is exactly zero, so the rows
    of dW_x stay finite."""
    rng = np.random.Generator(np.random.PCG64(K))
    wl = _trees(K, inputs, rng)
    for row, d, v in ((0, 3, HUGE), (wl.n_x // 2, 7, -HUGE), (wl.n_x - 1, 19, HUGE)):
        wl.X[row, d] = v
    print("large inputs K=%d %s V=%d n_x=%d" % (K, inputs, wl.V, wl.n_x), flush=True)
    check(Batch(wl, ctx).run(), oracle_sharded(wl), ["h", "c", "loss", "dWx", "dU", "db", "dX"],
          1e-4, "large", floor=1.0)


@pytest.mark.parametrize("K", [40, 1200])
def test_infinite_inputs(ctx, K):
    rng = np.random.Generator(np.random.PCG64(K + 1))
    wl = _trees(K, "leaves", rng)
    wl.X[0, 3], wl.X[wl.n_x // 2, 7], wl.X[wl.n_x - 1, 19] = np.inf, -np.inf, np.inf
    print("infinite inputs K=%d V=%d" % (K, wl.V), flush=True)
    got, want = Batch(wl, ctx).run(), oracle_sharded(wl)
    check(got, want, ["h", "c", "loss", "dU", "db", "dX"], 1e-4, "infinite", floor=1.0)
    # inf times a gradient of zero: those rows of dW_x are NaN in any order of summation
    rest = [d for d in range(wl.D) if d not in (3, 7, 19)]
    check({"dWx": got["dWx"][rest]}, {"dWx": want["dWx"][rest]}, ["dWx"], 1e-4, "rest", floor=1.0)


def test_large_head_weights(ctx):
    """Logits and dL/dh of a large-vocabulary head with a class weight above
    bf16's range: the loss is large and finite."""
    rng = np.random.Generator(np.random.PCG64(3))
    wl = W.make_workload("head", [W.chain(5)] * 30, N=1, D=8, H=64, C=132, sigma=0.1, rng=rng,
                         inputs="all", labels="all")
    wl.Ws[5, 17] = HUGE
    wl.push_idx[wl.push_idx == 17] = 18
    wl.push_idx[3:] = -1          # three terms: their sum is in range too
    got, want = Batch(wl, ctx).run(backward=False), oracle_sharded(wl, backward=False)
    assert np.isfinite(want["loss"])
    check(got, want, ["h", "loss"], 1e-4, "head", floor=1.0)


@pytest.mark.parametrize("H", [64, 320, 512])
def test_large_recurrent_weights(ctx, monkeypatch, H):
    """The level loop holds U as parts: a weight beyond their range saturates
    its unit's gate as on the level kernels."""
    rng = np.random.Generator(np.random.PCG64(H))
    wl = W.make_workload("u", [W.chain(int(n)) for n in rng.integers(2, 9, size=20)], N=1, D=8, H=H,
                         C=5, sigma=0.1, rng=rng, inputs="all", labels="all")
    wl.U[3, 2], wl.U[H - 1, 2 * H + 5], wl.U[9, 3 * H + 1] = HUGE, -HUGE, HUGE
    want = oracle_sharded(wl, backward=False)
    for mode in ("0", "1"):
        monkeypatch.setenv("CAVS_XCD_LOOP", mode)
        print("large U H=%d loop=%s" % (H, mode), flush=True)
        check(Batch(wl, ctx).run(backward=False), want, ["h", "c", "loss"], 1e-4, "u" + mode,
              floor=1.0)
