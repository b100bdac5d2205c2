"""One fp32 workspace for many batches: the size asked for one batch serves any
other with as many vertices and input rows, whatever its levels are."""
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


@pytest.mark.parametrize("H", [64, 512])
def test_workspace_of_a_shallower_batch(ctx, monkeypatch, H):
    monkeypatch.setenv("CAVS_XCD_LOOP", "1")
    make = lambda graphs: W.make_workload("ws", graphs, N=2, D=8, H=H, C=5, sigma=0.1,
                                          rng=np.random.Generator(np.random.PCG64(H)),
                                          inputs="all", labels="all")
    flat = make([W.complete_tree(2)] * 90)              # one level above the leaves
    deep = make([W.left_branching_tree(5)] * 30)        # four, of 30 each
    assert flat.V == deep.V and flat.n_x == deep.n_x
    a, b = Batch(flat, ctx), Batch(deep, ctx)
    a.schedule()
    b.schedule()
    b.alloc()
    nbytes = B.workspace_bytes(a.params, a.sched)
    assert nbytes < b.ws.numel()
    b.ws = torch.empty(nbytes, dtype=torch.uint8, device=b.dev)
    print("workspace of a flat batch: %d bytes, H=%d V=%d" % (nbytes, H, deep.V), flush=True)
    check_fp32(b.run(), oracle_sharded(deep), oracle_sharded(deep, precision="f32"), KEYS, "ws")
