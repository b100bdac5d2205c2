"""Two contexts on two streams of one device, both with batches that take the
level loop: enqueued side by side from one thread and from two, no loop gives
up (cavs_sync reports it if one does) and every result is what the batch gives
alone, bit for bit.  A pass captured beside another context's use gives the
same, replayed while the other one is idle."""
import threading

import numpy as np
import pytest
import torch

from paper_1712_04048_amd import binding as B
from paper_1712_04048_amd import workloads as W
from paper_1712_04048_amd.runner import Batch

pytestmark = pytest.mark.gpu

REPS = 20


def _pair():
    out = []
    for H, N, seed in ((256, 1, 1), (512, 2, 2)):
        rng = np.random.Generator(np.random.PCG64(seed))
        make = W.chain if N == 1 else (lambda n: W.random_split_tree(n, rng))
        wl = W.make_workload("pair", [make(int(n)) for n in rng.integers(8, 30, size=40)], N=N, D=16,
                             H=H, C=5, sigma=0.1, rng=rng, inputs="all" if N == 1 else "leaves",
                             labels="all")
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            b = Batch(wl, B.Context(0, stream))
            b.run()
        want = b.results()
        out.append((b, stream, want))
    torch.cuda.synchronize()
    return out


def _check(b, want):
    for k, v in b.results().items():
        assert np.array_equal(np.asarray(v), np.asarray(want[k])), k


def _close(pair):
    torch.cuda.synchronize()
    for b, _, _ in pair:
        b.ctx.close()


def test_side_by_side(monkeypatch):
    monkeypatch.setenv("CAVS_XCD_LOOP", "1")
    pair = _pair()
    print("two contexts, one thread: V = %s" % [b.wl.V for b, _, _ in pair], flush=True)
    for _ in range(REPS):
        for b, _, _ in pair:
            b.forward()
        for b, _, _ in pair:
            b.backward()
    for b, _, want in pair:
        b.ctx.sync()
        _check(b, want)
    _close(pair)


def test_two_threads(monkeypatch):
    monkeypatch.setenv("CAVS_XCD_LOOP", "1")
    pair = _pair()
    errors = []

    def work(b, stream):
        try:
            torch.cuda.set_device(0)
            with torch.cuda.stream(stream):
                for _ in range(REPS):
                    b.step()
                b.ctx.sync()
        except Exception as e:   # reported by the main thread
            errors.append(e)

    print("two contexts, two threads", flush=True)
    threads = [threading.Thread(target=work, args=(b, s)) for b, s, _ in pair]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for b, _, want in pair:
        _check(b, want)
    _close(pair)


def test_capture_beside_another_context(monkeypatch):
    monkeypatch.setenv("CAVS_XCD_LOOP", "1")
    pair = _pair()
    (b, stream, want), (other, _, other_want) = pair
    print("capture beside another context", flush=True)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        b.forward()
        b.backward()
    for _ in range(3):
        other.forward()
        other.backward()
        other.ctx.sync()
        g.replay()
        torch.cuda.synchronize()
        b.ctx.sync()
        _check(b, want)
        _check(other, other_want)
    _close(pair)


def test_context_after_context(monkeypatch):
    """A context's loops follow those of one that is gone."""
    monkeypatch.setenv("CAVS_XCD_LOOP", "1")
    for _ in range(3):
        pair = _pair()
        for b, _, want in pair:
            b.forward()
            b.backward()
        for b, _, want in pair:
            b.ctx.sync()
            _check(b, want)
        _close(pair)
