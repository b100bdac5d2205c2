"""GPU parity of the level products at hidden widths that are not multiples
of 256 (short last shares of the split-K contraction, ragged column tiles of
the lazy products) and at three and four child slots, over tree and graph
inputs: levels on both sides of the split-K / tile lines, inputs at every
vertex (the forget columns of dW_x and dX are sums over slots)."""
import numpy as np
import pytest
import torch

import oracle
from parity import check, check_fp32, oracle_sharded
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


def _graphs(kind, N, K, rng):
    if kind == "chain":
        return [W.chain(int(n)) for n in rng.integers(1, 7, size=K)]
    if kind == "dag":
        return [W.random_dag(int(n), N, rng) for n in rng.integers(2, 9, size=K)]
    if kind == "nary":
        return [W.nary_tree(int(n), N, rng) for n in rng.integers(1, 9, size=K)]
    return [W.random_split_tree(int(n), rng) for n in rng.integers(1, 9, size=K)]


# (H, N, kind, K, D, inputs): K graphs give a first level of K or fewer positions
CASES = [(64, 1, "chain", 300, 20, "all"), (64, 2, "split", 1700, 12, "leaves"),
         (192, 2, "split", 460, 36, "all"), (320, 2, "split", 37, 100, "all"),
         (320, 2, "split", 330, 68, "all"), (320, 1, "chain", 330, 4, "all"),
         (448, 2, "split", 20, 300, "leaves"), (576, 1, "chain", 150, 8, "all"),
         (576, 2, "split", 130, 132, "leaves"), (192, 3, "nary", 500, 28, "all"),
         (320, 4, "nary", 320, 64, "leaves"), (256, 3, "nary", 30, 12, "all"),
         (64, 4, "nary", 40, 8, "all"), (320, 2, "dag", 330, 12, "all"),
         (192, 4, "dag", 40, 8, "leaves"), (128, 1, "dag", 50, 8, "all"),
         (512, 3, "dag", 210, 8, "all")]


@pytest.mark.parametrize("H,N,kind,K,D,inputs", CASES)
def test_level_products(ctx, H, N, kind, K, D, inputs):
    rng = np.random.Generator(np.random.PCG64(1000 * H + 10 * K + N))
    wl = W.make_workload("widths", _graphs(kind, N, K, rng), N=N, D=D, H=H, C=5,
                         sigma=0.3 if H <= 128 else 0.05, rng=rng, inputs=inputs, labels="all",
                         shuffle_ids=True, dag=kind == "dag")
    wl.b[:] = (0.1 * rng.standard_normal(wl.b.shape)).astype(np.float32)
    print("widths H=%d N=%d %s V=%d" % (H, N, kind, wl.V), flush=True)
    b = Batch(wl, ctx)
    got = b.run()
    check_fp32(got, oracle_sharded(wl), oracle_sharded(wl, precision="f32"), KEYS, "widths")
    # inference computes the same states
    assert np.array_equal(b.run_infer()["h"], got["h"])


@pytest.mark.parametrize("H,N,K,D,inputs", [
    (320, 2, 70, 36, "all"), (320, 1, 90, 36, "all"), (192, 2, 64, 36, "all"),
    (128, 2, 720, 36, "all"), (576, 2, 300, 36, "leaves"), (64, 2, 43, 4, "leaves"),
    (192, 2, 65, 132, "leaves"),
    (128, 2, 8100, 4, "leaves"), (320, 1, 3300, 4, "all")])
def test_level_products_bf16(ctx, H, N, K, D, inputs):
    """Shallow graphs (bf16 rounding points differ little), element by
    element at the 10% floor against the bf16-emulating oracle; 720 cherries
    at H = 128 put the backward on tiles, the forward on two-row split-K, 300
    at 576 both on tiles, 8100 cherries and 3300 chains the forward on 128-row
    tiles, the last one ragged; inputs at leaves only take the pull product
    with the leaf cells in its epilogue, at depths that are no multiple of its
    32-deep chunk."""
    rng = np.random.Generator(np.random.PCG64(H + K + N))
    graphs = [W.complete_tree(2)] * K if N == 2 else [W.chain(3)] * K
    wl = W.make_workload("widths_bf16", graphs, prec=W.PREC_BF16, N=N, D=D, H=H, C=5, sigma=0.1,
                         rng=rng, inputs=inputs, labels="all")
    print("widths bf16 H=%d N=%d D=%d %s V=%d" % (H, N, D, inputs, wl.V), flush=True)
    check(Batch(wl, ctx).run(), oracle_sharded(wl, bf16=True), KEYS, 2e-2, "widths_bf16", floor=0.1)


# inputs at leaves only (three gate blocks) and at every vertex (four), the
# 64 x 64 tiles filled to 1 020 workgroups and the 128 x 128 tiles above that
@pytest.mark.parametrize("H,N,K,D,inputs", [
    (128, 2, 6500, 260, "leaves"), (128, 2, 8100, 260, "leaves"), (320, 1, 3300, 452, "all")])
def test_dx_bf16(ctx, H, N, K, D, inputs):
    """bf16 dX on both sides of the line between its tiles, the last tile
    ragged in rows and columns; shallow graphs at the bar of the bf16 level
    products above."""
    rng = np.random.Generator(np.random.PCG64(H + K + D))
    graphs = [W.complete_tree(2)] * K if N == 2 else [W.chain(3)] * K
    wl = W.make_workload("dx_bf16", graphs, prec=W.PREC_BF16, N=N, D=D, H=H, C=5, sigma=0.1,
                         rng=rng, inputs=inputs, labels="all")
    print("dx bf16 H=%d N=%d D=%d %s V=%d" % (H, N, D, inputs, wl.V), flush=True)
    check(Batch(wl, ctx).run(), oracle_sharded(wl, bf16=True), KEYS, 2e-2, "dx_bf16", floor=0.1)


@pytest.mark.parametrize("prec,H,D", [(W.PREC_BF16, 64, 36), (W.PREC_BF16, 320, 4),
                                      (W.PREC_FP32, 512, 36)])
def test_one_level_in_a_poisoned_workspace(ctx, prec, H, D):
    """Single vertices only: no level product runs, so the pull product's
    launches alone must write whatever they read of the workspace (the zero
    row past a ragged depth or the last vertex)."""
    rng = np.random.Generator(np.random.PCG64(H + D))
    K = 2100 if prec == W.PREC_FP32 else 70    # fp32: enough rows for the split pull product
    wl = W.make_workload("one_level", [W.chain(1)] * K, prec=prec, N=1, D=D, H=H, C=5, sigma=0.1,
                         rng=rng, inputs="all", labels="all")
    b = Batch(wl, ctx)
    b.schedule()
    b.alloc()
    b.ws.fill_(255)   # NaN in fp32 and bf16
    b.ws_infer = torch.full_like(b.ws, 255)
    got = b.run()
    if prec == W.PREC_FP32:
        check_fp32(got, oracle_sharded(wl), oracle_sharded(wl, precision="f32"), KEYS, "one_level")
    else:
        check(got, oracle_sharded(wl, bf16=True), KEYS, 2e-2, "one_level", floor=0.1)
    assert np.array_equal(b.run_infer()["h"], got["h"])
