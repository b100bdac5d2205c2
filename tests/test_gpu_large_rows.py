"""Gradients where an operand holds more than 2^31 elements: the row offsets of
the lazy products pass 32 bits.  X is made that large (rows nobody pulls cost
nothing but memory), a few hundred vertices pull rows at both of its ends, and
the rest of the problem is small, so the oracle evaluates it on the pulled rows
alone.  One, two, three and four child slots, and Tree-FC; the bar is that of
parity.check_fp32."""
import numpy as np
import pytest
import torch

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


@pytest.mark.parametrize("cell,N,inputs", [("lstm", 1, "all"), ("lstm", 2, "leaves"),
                                           ("lstm", 3, "all"), ("lstm", 4, "leaves"),
                                           ("fc", 2, "leaves")])
def test_more_than_2_31_elements_of_x(ctx, cell, N, inputs):
    rng = np.random.Generator(np.random.PCG64(N))
    make = {1: W.chain, 2: lambda n: W.random_split_tree(n, rng)}.get(
        N, lambda n: W.nary_tree(n, N, rng))
    D = 64 if cell == "fc" else 8
    wl = W.make_workload("rows", [make(int(n)) for n in rng.integers(2, 12, size=30)],
                         cell=W.CELL_TREE_FC if cell == "fc" else W.CELL_TREE_LSTM, N=N, D=D, H=64,
                         C=5, sigma=0.1, rng=rng, inputs=inputs, labels="all")
    n_x = (1 << 31) // D + 64
    assert n_x * D > 1 << 31
    row = np.arange(wl.n_x, dtype=np.int64)
    row[1::2] = n_x - 1 - row[1::2]          # every other pulled row at the far end
    b = Batch(wl, ctx)
    dev = b.dev
    X = torch.empty(n_x, D, dtype=torch.float32, device=dev)
    at = torch.from_numpy(row).to(dev)
    X[at] = b.X
    b.X = X
    pull = np.where(wl.pull_idx >= 0, row[np.maximum(wl.pull_idx, 0)], -1).astype(np.int32)
    print("large rows %s N=%d V=%d n_x=%d D=%d" % (cell, N, wl.V, n_x, D), flush=True)
    b.sched = B.schedule(ctx, b.child, b.parent, torch.from_numpy(pull).to(dev), b.push_idx,
                         n_x=n_x, n_push=wl.n_push)
    b.alloc()
    dX = b.grads["dX"] = torch.empty(n_x, D, dtype=torch.float32, device=dev)
    b.forward()
    b.backward()
    ctx.sync()
    b.grads["dX"] = dX[at]
    assert int(torch.count_nonzero(dX)) <= wl.n_x * D    # the rows nobody pulls are zero
    check_fp32(b.results(), oracle_sharded(wl), oracle_sharded(wl, precision="f32"), KEYS,
               "large_rows")
