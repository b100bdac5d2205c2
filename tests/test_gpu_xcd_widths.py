"""The XCD-local level loop at every kind of width and slot count it takes:
forced on (CAVS_XCD_LOOP=1) and off, over batches that give an XCD no row, a
few rows and several 16-row tiles of a level; a second backward after one
forward (the loop's barrier words carry on) gives the same gradients bit for
bit.  Both ways evaluate the same definitions in fp32 with sums in another
order: 1e-5 of each tensor's largest value (the tolerance of the loop's other
tests)."""
import numpy as np
import pytest

from parity import check, oracle_sharded
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


CASES = [(64, 2, 1, 40), (64, 1, 250, 12), (128, 4, 30, 20), (192, 3, 9, 30), (192, 2, 230, 9),
         (256, 3, 120, 12), (320, 1, 200, 10), (320, 2, 20, 30), (448, 2, 3, 50), (512, 2, 190, 12),
         (512, 1, 17, 25), (256, 4, 240, 8)]


@pytest.mark.parametrize("H,N,K,size", CASES)
def test_loop_on_and_off(ctx, monkeypatch, H, N, K, size):
    rng = np.random.Generator(np.random.PCG64(H + 10 * N + K))
    make = {1: lambda n: W.chain(n), 2: lambda n: W.random_split_tree(n, rng)}.get(
        N, lambda n: W.nary_tree(n, N, rng))
    wl = W.make_workload("xcd", [make(int(n)) for n in rng.integers(1, size + 1, size=K)], N=N,
                         D=20, H=H, C=5, sigma=0.1 if H <= 256 else 0.05, rng=rng,
                         inputs="all" if N != 2 else "leaves", labels="all", shuffle_ids=True)
    print("xcd widths H=%d N=%d K=%d V=%d" % (H, N, K, wl.V), flush=True)
    out = {}
    for mode in ("0", "1"):
        monkeypatch.setenv("CAVS_XCD_LOOP", mode)
        b = Batch(wl, ctx)
        out[mode] = b.run()
    b.backward()
    ctx.sync()
    again = b.results()
    for k, v in out["0"].items():
        scale = max(float(np.abs(v).max()), 1e-30)
        assert float(np.abs(out["1"][k] - v).max()) <= 1e-5 * scale, k
        assert np.array_equal(np.asarray(again[k]), np.asarray(out["1"][k])), k


@pytest.mark.parametrize("H,N,K,size", [(320, 2, 30, 6), (576, 2, 140, 3), (576, 1, 130, 3),
                                        (832, 2, 9, 6), (1024, 1, 8, 6), (1024, 2, 20, 4)])
def test_loop_bf16(ctx, monkeypatch, H, N, K, size):
    """bf16 widths on one and two unit tiles per workgroup (the latter from
    512 units up, the last wavefronts short of chunks), one and two row tiles
    per level: shallow graphs (bf16 rounding points differ little), element by
    element at the 10% floor against the bf16-emulating oracle."""
    rng = np.random.Generator(np.random.PCG64(H + 10 * N + K))
    make = W.chain if N == 1 else lambda n: W.random_split_tree(n, rng)
    wl = W.make_workload("xcd_bf16", [make(int(n)) for n in rng.integers(2, size + 1, size=K)],
                         prec=W.PREC_BF16, N=N, D=36, H=H, C=5, sigma=0.05, rng=rng,
                         inputs="all" if N == 1 else "leaves", labels="all", shuffle_ids=True)
    print("xcd bf16 H=%d N=%d K=%d V=%d" % (H, N, K, wl.V), flush=True)
    want = oracle_sharded(wl, bf16=True)
    for mode in ("0", "1"):
        monkeypatch.setenv("CAVS_XCD_LOOP", mode)
        check(Batch(wl, ctx).run(), want, KEYS, 2e-2, "xcd_bf16_%s" % mode, floor=0.1)
