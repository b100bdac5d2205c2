"""GPU parity of the split fp32 products (three bf16 parts per operand): the
lazy weight gradients and the large-vocabulary head, at sizes where they can
go wrong (one short chunk, ragged tiles on both sides, several row-offset
segments, one split and many), and operands over a wide range of magnitudes.

The oracle comparisons carry the fp32 bar of parity.check_fp32.  The range
tests scale weights and inputs by powers of two, which an exact split (and
fp32) carries through without any new rounding: the gradients of the scaled
problem equal the scaled gradients bit for bit."""
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


@pytest.mark.parametrize("H,n_pull_min", [(128, 0), (512, 1921)])
def test_power_of_two_scaling_of_the_input_side(ctx, H, n_pull_min):
    """As above with dX as well (a factor 2^k on W_x's row d is one on dX's
    column d), and with more rows: from 1 921 pulled rows at H = 512 the pull
    product is a split product too."""
    rng = np.random.Generator(np.random.PCG64(H))
    trees = [W.random_split_tree(int(n), rng) for n in rng.integers(2, 30, size=40 if H < 512 else 80)]
    wl = W.make_workload("scale", trees, N=2, D=64, H=H, C=5, sigma=0.05, rng=rng, inputs="all",
                         labels="all")
    assert int((wl.pull_idx >= 0).sum()) >= n_pull_min
    a = Batch(wl, ctx).run()
    k = rng.integers(-40, 41, size=wl.D)
    f = (2.0 ** k).astype(np.float32)
    wl.X = wl.X * f
    wl.Wx = wl.Wx / f[:, None]
    b = Batch(wl, ctx).run()
    for key in ("h", "c", "dU", "db"):
        assert np.array_equal(a[key], b[key]), key
    f = f.astype(np.float64)
    assert np.array_equal(a["dWx"] * f[:, None], b["dWx"])
    assert np.array_equal(a["dX"] / f, b["dX"])


def test_power_of_two_scaling_of_the_head(ctx):
    """W_s so small that every logit is its bias bit for bit: a factor 2^k on
    row j of W_s then leaves loss, dW_s and db_s as they are, and dL/dh's
    unit j, with the gradients of its gates' columns, is 2^k times what it
    was (single vertices: no unit meets another behind the head)."""
    rng = np.random.Generator(np.random.PCG64(7))
    wl = W.make_workload("scale_head", [W.chain(1)] * 300, N=1, D=8, H=64, C=260, sigma=0.1,
                         rng=rng, inputs="all", labels="all")
    wl.bs[:] = rng.uniform(0.5, 1.0, wl.C).astype(np.float32)
    wl.Ws = wl.Ws * np.float32(2.0 ** -50)
    a = Batch(wl, ctx).run()
    f = (2.0 ** rng.integers(-10, 11, size=wl.H)).astype(np.float32)
    wl.Ws = wl.Ws * f[:, None]
    b = Batch(wl, ctx).run()
    for key in ("h", "loss", "dWs", "dbs"):
        assert np.array_equal(a[key], b[key]), key
    cols = np.tile(f.astype(np.float64), 4)   # the gate blocks' columns
    assert np.any(a["db"] != 0)
    assert np.array_equal(a["db"] * cols, b["db"])
    assert np.array_equal(a["dWx"] * cols, b["dWx"])


def test_head_over_a_wide_range_of_columns(ctx):
    """Columns of W_s from 2^-40 to 2^3 times their usual size."""
    rng = np.random.Generator(np.random.PCG64(8))
    wl = W.make_workload("wide_head", [W.chain(5)] * 60, N=1, D=12, H=128, C=260, sigma=0.1,
                         rng=rng, inputs="all", labels="all")
    wl.Ws = wl.Ws * (2.0 ** rng.integers(-40, 4, size=wl.C)).astype(np.float32)
    check_fp32(Batch(wl, ctx).run(), oracle_sharded(wl), oracle_sharded(wl, precision="f32"), KEYS,
               "wide_head")


@pytest.mark.parametrize("K", [1024, 1049])
def test_dw_on_both_sides_of_a_workgroup_per_cu(ctx, K):
    """Tree-FC dW at H = 256 (eight tiles over both slots): 32 chunks make 256
    workgroups of one chunk each, 33 take two each, the last one a ragged one."""
    rng = np.random.Generator(np.random.PCG64(K))
    wl = W.make_workload("fc_dw", [W.complete_tree(2)] * K, cell=W.CELL_TREE_FC, loss=W.LOSS_L2, N=2,
                         D=256, H=256, sigma=0.05, rng=rng, inputs="leaves", labels="root")
    keys = ["h", "loss", "dU", "db", "dX"]
    check_fp32(Batch(wl, ctx).run(), oracle_sharded(wl), oracle_sharded(wl, precision="f32"), keys,
               "fc_dw")
