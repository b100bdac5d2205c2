"""GPU parity of the split fp32 products (three bf16 parts per operand): the
lazy weight gradients and the large-vocabulary head, at sizes where they can
go wrong (one short chunk, ragged tiles on both sides, several row-offset
segments, one split and many), and operands over a wide range of magnitudes.

The oracle comparison carries the fp32 bar of parity.check_fp32.  The range
test scales the weights' rows and the inputs by powers of two, which an exact
split (and fp32) carries through without any new rounding: the gradients of
the scaled problem equal the scaled gradients bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from parity import check_fp32, oracle_sharded
from paper_1712_04048_amd import binding as B
from paper_1712_04048_amd import workloads as W
from paper_1712_04048_amd.runner import Batch

pytestmark = pytest.mark.gpu

KEYS = ["h", "c", "loss", "dWx", "dU", "db", "dWs", "dbs", "dX"]


@pytest.fixture(scope="module")
def ctx():
    c = B.Context(0)
    yield c
    c.close()


# K chains of length L: vertices, classes, H, D
@pytest.mark.parametrize("K,L,C,H,D", [(1, 2, 20, 64, 4), (3, 43, 260, 64, 132), (2, 33, 1028, 192, 8),
                                       (40, 40, 4100, 64, 12), (5, 13, 128, 128, 128),
                                       (9, 15, 10244, 64, 4), (3, 11, 16388, 64, 4)])
def test_head_and_chain_gradients(ctx, K, L, C, H, D):
    rng = np.random.Generator(np.random.PCG64(K * 100 + C))
    wl = W.make_workload("x3", [W.chain(L)] * K, N=1, D=D, H=H, C=C, sigma=0.1, rng=rng,
                         inputs="all", labels="all")
    wl.push_idx[::5] = -1          # unlabelled vertices too
    wl.bs[:] = (0.1 * rng.standard_normal(C)).astype(np.float32)
    print("x3 V=%d C=%d H=%d D=%d" % (wl.V, C, H, D), flush=True)
    check_fp32(Batch(wl, ctx).run(), oracle_sharded(wl), oracle_sharded(wl, precision="f32"), KEYS,
               "x3_head")


def test_power_of_two_scaling_is_exact(ctx):
    """dX scales with the rows of W_x, dW_x with the columns of X: a factor
    2^k on input dimension d in X and 2^-k in W_x leaves every state as it is
    and multiplies dW_x's row d by 2^k."""
    rng = np.random.Generator(np.random.PCG64(5))
    trees = [W.random_split_tree(int(n), rng) for n in rng.integers(2, 30, size=40)]
    wl = W.make_workload("scale", trees, N=2, D=64, H=128, C=5, sigma=0.1, rng=rng, inputs="all",
                         labels="all")
    a = Batch(wl, ctx).run()
    k = rng.integers(-40, 41, size=wl.D)
    f = (2.0 ** k).astype(np.float32)
    wl.X = wl.X * f
    wl.Wx = wl.Wx / f[:, None]
    b = Batch(wl, ctx).run()
    assert np.array_equal(a["h"], b["h"])
    assert np.array_equal(a["dU"], b["dU"])
    assert np.array_equal(a["dWx"] * f[:, None].astype(np.float64), b["dWx"])
