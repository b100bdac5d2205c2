"""The work this library is measured on.

A user of the library has one thing done for every minibatch: its graphs are
scheduled (cavs_schedule), and the vertex function runs over them -- forward
and backward when training, forward alone when serving -- through the Python
binding of the C ABI.  The cases are that work for the recurrent structures
the vertex functions exist for (parse trees, sentences, complete trees, wider
trees, graphs with shared vertices), from batches where launches and latency
decide to the largest ones, in both precisions and with both kinds of head.

Every batch is new work for the library: a pass schedules the batch again and
keeps nothing of an earlier one.
"""
import math

import numpy as np
import torch

from paper_1712_04048_amd import binding as B
from paper_1712_04048_amd import workloads as W

LSTM, FC = "lstm", "fc"

# Defaults of a case; a case names what differs.
#   kind    train: schedule + forward + backward; infer: schedule + cavs_infer;
#           schedule: the schedule alone
#   graph   split: random binary trees; sst: the same with parse-tree sizes;
#           chain; complete: complete binary trees; left: half left-branching
#           trees, half random; nary: 2..N children; dag: shared vertices
#   K graphs, lo..hi leaves (vertices for chains and dags) in each
#   N child slots, D inputs, H hidden units, C classes (0: L2 against targets)
DEFAULTS = dict(kind="train", cell=LSTM, bf16=False, graph="sst", K=1, lo=2, hi=56, N=2, D=64,
                H=64, C=5, inputs="leaves", labels="all", sigma=0.05, dag=False)


def _case(name, **kw):
    c = dict(DEFAULTS)
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # A handful of small trees: interactive use and tests of a model; launches and latency.
        _case("tiny_train", graph="split", K=8, lo=4, hi=16, labels="root", sigma=0.1),
        # The headline: Tree-LSTM training over a sentiment-treebank batch, a loss at every vertex.
        _case("sst_train", K=256, D=300, H=512),
        # A serving request: 16 parsed sentences, states and loss only.
        _case("sst_infer_16", kind="infer", K=16, D=300, H=512),
        # A small training batch at a width between the usual ones, inputs at every vertex,
        # half the trees as deep as they have leaves.
        _case("mixed_trees_train", graph="left", K=37, lo=1, hi=40, D=100, H=320, inputs="all"),
        # Sentence classification with variable-length LSTMs: up to 100 dependent steps.
        _case("varlstm_train", graph="chain", K=64, lo=10, hi=100, N=1, D=512, H=512,
              inputs="all", labels="root"),
        # Tree-FC over complete trees of 256 leaves.
        _case("treefc_train", cell=FC, graph="complete", K=64, lo=256, hi=256, D=512, H=512, C=0,
              labels="root"),
        # A wide bf16 Tree-LSTM over deep trees: the largest batch.
        _case("deep_bf16_train", bf16=True, graph="left", K=256, lo=32, hi=128, D=300, H=1024,
              sigma=0.03),
        # bf16 serving of many parsed sentences at once.
        _case("sst_bf16_infer", kind="infer", bf16=True, K=1024, D=300, H=512),
        # Graph-structured cells: vertices read by several others, four slots.
        _case("dag_train", graph="dag", K=160, lo=10, hi=40, N=4, D=300, H=512, dag=True),
        # Child-sum trees with three slots and a word at every vertex (dependency trees).
        _case("nary_train", graph="nary", K=61, lo=3, hi=40, N=3, D=300, H=256, inputs="all"),
        # A language model: a 10 000-word softmax at every step of every sentence.
        _case("lm_train", graph="chain", K=64, lo=10, hi=60, N=1, D=512, H=512, C=10000,
              inputs="all"),
        # Scheduling alone of a forest of some 74 000 vertices (many sentences at once).
        _case("forest_schedule", kind="schedule", K=2000, D=4, H=64),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(case):
    """Rough number of vertices of a case, before its graphs are drawn."""
    g = case["graph"]
    mean = 19.0 if g == "sst" else 0.5 * (case["lo"] + case["hi"])
    per = mean if g in ("chain", "dag") else 1.6 * mean if g == "nary" else 2 * mean - 1
    return case["K"] * per


def _cost(case):
    """Rough floating-point work of a case, in TFLOP."""
    H, V = case["H"], _size(case)
    per = 6 * H * H if case["cell"] == FC else 30 * H * H + 18 * case["D"] * H
    return V * (per + (6 * H * case["C"] if case["C"] > 16 else 0)) * 1e-12


def draw(rng):
    """One more case of the ranges the listed ones stand for."""
    while True:
        what = rng.choice(["trees", "trees", "small", "chains", "fc", "bf16", "infer", "dag",
                           "nary", "lm", "schedule"])
        H = 64 * _log(rng, 1, 16)
        D = 4 * _log(rng, 2, 128)
        inputs = rng.choice(["leaves", "all"])
        lo = rng.randint(1, 10)
        hi = lo + _log(rng, 4, 60)
        cap = 0.08
        if what == "trees":
            c = _case(None, graph=rng.choice(["sst", "split", "left"]), K=_log(rng, 4, 400),
                      lo=lo, hi=hi, D=D, H=H, inputs=inputs, labels=rng.choice(["all", "root"]))
        elif what == "small":
            c = _case(None, graph="split", K=_log(rng, 1, 32), lo=lo, hi=lo + 12, D=64,
                      H=64 * rng.randint(1, 4), labels="root", sigma=0.1)
        elif what == "chains":
            c = _case(None, graph="chain", K=_log(rng, 1, 200), lo=lo, hi=2 * hi, N=1, D=D, H=H,
                      inputs="all", labels=rng.choice(["all", "root"]))
        elif what == "fc":
            if rng.random() < 0.5:
                leaves = 1 << rng.randint(4, 9)
                c = _case(None, cell=FC, graph="complete", K=_log(rng, 4, 100), lo=leaves,
                          hi=leaves, D=H, H=H, C=0, labels="root")
            else:
                c = _case(None, cell=FC, graph="split", K=_log(rng, 4, 400), lo=lo, hi=hi, D=H,
                          H=H, C=rng.choice([0, 5]), labels=rng.choice(["all", "root"]))
        elif what == "bf16":
            c = _case(None, bf16=True, graph=rng.choice(["sst", "left"]), K=_log(rng, 16, 300),
                      lo=lo, hi=2 * hi, D=D, H=H, inputs=inputs)
            cap = 1.0
        elif what == "infer":
            c = _case(None, kind="infer", bf16=rng.random() < 0.5, graph="sst",
                      K=_log(rng, 1, 1200), D=D, H=H, inputs=inputs)
            cap = 0.2
        elif what == "dag":
            c = _case(None, graph="dag", K=_log(rng, 4, 160), lo=lo + 1, hi=lo + 30,
                      N=rng.randint(1, 4), D=D, H=H, inputs=inputs, dag=True)
        elif what == "nary":
            c = _case(None, graph="nary", K=_log(rng, 4, 160), lo=lo, hi=hi, N=rng.randint(3, 4),
                      D=D, H=H, inputs=inputs)
        elif what == "lm":
            c = _case(None, graph="chain", K=_log(rng, 4, 64), lo=lo, hi=hi, N=1, D=D, H=H,
                      C=4 * _log(rng, 10, 2500), inputs="all")
            cap = 0.12
        else:
            c = _case(None, kind="schedule", graph=rng.choice(["sst", "split", "left"]),
                      K=_log(rng, 4, 2000), lo=lo, hi=hi, D=4, H=64)
        if _size(c) <= 80000 and (c["kind"] == "schedule" or _cost(c) <= cap):
            c["sigma"] = 0.1 if c["H"] <= 128 else 0.05 if c["H"] <= 512 else 0.03
            return c


def _workload(case, seed):
    """The batch's graphs, inputs and parameters.

    The graphs themselves are the case's (so that every seed's outputs have
    the same sizes); their order in the batch, and with it every index, the
    inputs, labels and parameters come from the seed.
    """
    rng = np.random.Generator(np.random.PCG64(0))
    K, lo, hi, N = case["K"], case["lo"], case["hi"], case["N"]
    g = case["graph"]
    sizes = W.sst_leaf_counts(K, rng) if g == "sst" else rng.integers(lo, hi + 1, size=K)
    if g == "chain":
        graphs = [W.chain(int(n)) for n in sizes]
    elif g == "complete":
        graphs = [W.complete_tree(int(n)) for n in sizes]
    elif g == "left":
        graphs = [W.left_branching_tree(int(n)) if k < K // 2
                  else W.random_split_tree(int(n), rng) for k, n in enumerate(sizes)]
    elif g == "nary":
        graphs = [W.nary_tree(int(n), N, rng) for n in sizes]
    elif g == "dag":
        graphs = [W.random_dag(int(n), N, rng, window=10) for n in sizes]
    else:
        graphs = [W.random_split_tree(int(n), rng) for n in sizes]
    rng = np.random.Generator(np.random.PCG64(int(seed)))
    graphs = [graphs[k] for k in rng.permutation(K)]
    wl = W.make_workload("case", graphs, cell=W.CELL_TREE_FC if case["cell"] == FC
                         else W.CELL_TREE_LSTM,
                         prec=W.PREC_BF16 if case["bf16"] else W.PREC_FP32,
                         loss=W.LOSS_CE if case["C"] else W.LOSS_L2, N=N, D=case["D"],
                         H=case["H"], C=case["C"], sigma=case["sigma"], rng=rng,
                         inputs=case["inputs"], labels=case["labels"], dag=case["dag"])
    # a model in use has biases
    wl.b[:] = (0.1 * rng.standard_normal(wl.b.shape)).astype(np.float32)
    if case["C"]:
        wl.bs[:] = (0.1 * rng.standard_normal(wl.bs.shape)).astype(np.float32)
    return wl


def prepare(case, seed):
    """The batch and the model on the GPU, and the buffers a program keeps for them."""
    wl = _workload(case, seed)
    ctx = B.Context(0)
    dev = ctx.torch_device

    def i32(a):
        return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(dev)

    def f32(a):
        return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(dev) \
            if a.size else None

    s = dict(kind=case["kind"], ctx=ctx, n_x=wl.n_x, n_push=wl.n_push,
             child=i32(wl.child.reshape(wl.V, wl.N)), parent=None if wl.dag else i32(wl.parent),
             pull=i32(wl.pull_idx), push=i32(wl.push_idx))
    s["sched"] = B.alloc_schedule(ctx, wl.V, wl.N, wl.n_x)
    if case["kind"] == "schedule":
        return s
    ce, lstm = wl.loss == W.LOSS_CE, wl.cell == W.CELL_TREE_LSTM
    s["X"], s["Y"] = f32(wl.X), None if ce else f32(wl.Y)
    p = s["params"] = B.Params(cell=wl.cell, prec=wl.prec, loss=wl.loss, D=wl.D, H=wl.H, N=wl.N,
                               C=wl.C if ce else 0, Wx=f32(wl.Wx) if lstm else None, U=f32(wl.U),
                               b=f32(wl.b), Ws=f32(wl.Ws) if ce else None,
                               bs=f32(wl.bs) if ce else None)
    _schedule(s)
    f = dict(dtype=torch.float32, device=dev)
    nbytes = (B.workspace_bytes if case["kind"] == "train" else B.infer_workspace_bytes)(
        p, s["sched"])
    s["ws"] = torch.empty(nbytes, dtype=torch.uint8, device=dev)
    s["h"] = torch.empty(wl.V, wl.H, **f)
    s["c"] = torch.empty(wl.V, wl.H, **f) if lstm else None
    s["loss"] = torch.empty(1, **f)
    if case["kind"] == "train":
        g = dict(dU=torch.empty_like(p.U), db=torch.empty_like(p.b),
                 dX=torch.empty(wl.n_x, wl.D, **f))
        if lstm:
            g["dWx"] = torch.empty_like(p.Wx)
        if ce:
            g["dWs"], g["dbs"] = torch.empty_like(p.Ws), torch.empty_like(p.bs)
        s["grads"] = g
    return s


def _schedule(s):
    B.run_schedule(s["ctx"], s["sched"], s["child"], s["parent"], s["pull"], s["push"],
                   n_x=s["n_x"], n_push=s["n_push"])


def run(s):
    """One minibatch: its schedule, then the forward and backward, or the forward alone."""
    _schedule(s)
    if s["kind"] == "schedule":
        t, raw = s["sched"].tensors, s["sched"].raw
        out = {k: t[k] for k in ("level", "order", "pos", "child_pos", "parent_pos", "pull_pos",
                                 "push_pos")}
        out["level_offsets"] = t["level_offsets"][: raw.T + 1]
        out["pull_list"] = t["pull_list"][: raw.n_pull]
        return out
    args = (s["ctx"], s["params"], s["sched"], s["X"], s["Y"], s["ws"])
    out = {"h": s["h"], "loss": s["loss"]}
    if s["c"] is not None:
        out["c"] = s["c"]
    if s["kind"] == "infer":
        B.infer(*args, s["h"], s["c"], s["loss"])
        return out
    B.forward(*args, s["h"], s["c"], s["loss"])
    B.backward(*args, s["grads"])
    out.update(s["grads"])
    return out


def _counts(case):
    """What work() needs of a case's graphs, taken from the graphs of seed 0."""
    wl = _workload(dict(case, D=4, H=64 if case["cell"] == FC else 4,
                        C=min(case["C"], 5)), 0)
    inner = (wl.child >= 0).any(axis=1)
    pulls = wl.pull_idx >= 0
    return dict(V=wl.V, links=int((wl.child >= 0).sum()), inner=int(inner.sum()),
                pulls=int(pulls.sum()), pull_leaf=int((pulls & ~inner).sum()),
                labelled=int((wl.push_idx >= 0).sum()))


def work(case):
    n = _counts(case)
    V, H, D, N, C = n["V"], case["H"], case["D"], case["N"], case["C"]
    graph = 4.0 * V * (N + 3)
    if case["kind"] == "schedule":
        # reads child, parent, pull, push; writes the nine arrays of the schedule
        return {"bytes": graph + 4.0 * V * (N + 6) + 4.0 * n["pulls"], "flops": 0.0}
    times = 3.0 if case["kind"] == "train" else 1.0     # backward: two products for each
    if case["cell"] == FC:
        flops = times * 2.0 * H * H * n["links"]
        weights, states, D = N * H * H + H, V * H, H
    else:
        # a pulling leaf has no use of the forget columns
        inp = 2.0 * D * H * (3 * n["pull_leaf"] + 4 * (n["pulls"] - n["pull_leaf"]))
        flops = times * (2.0 * H * H * (3 * n["inner"] + n["links"]) + inp)
        weights, states = 4 * H * (D + H + 1), 2 * V * H
    if C:
        flops += times * 2.0 * H * C * n["labelled"]
        weights += C * (H + 1)
    else:
        graph += 4.0 * n["labelled"] * H
    once = 4.0 * (weights + D * n["pulls"])
    return {"bytes": graph + once * (2 if case["kind"] == "train" else 1) + 4.0 * states,
            "flops": flops}


def tolerance(case):
    if case["kind"] == "schedule":
        return "exact"
    # Measured against exact(), times about four.  bf16: operands carry 8 bits,
    # sums and states are 32-bit (0.0029 at most).
    if case["bf16"]:
        return {"rel": 1.2e-2}
    # Graphs with shared vertices: every reader's gradient adds up level by
    # level, so the rounding of the states is amplified (2.5e-5).
    if case["dag"]:
        return {"rel": 1e-4}
    # 32-bit sums through many levels (3.0e-6).
    return {"rel": 1.2e-5}


# ---------------------------------------------------------------------------
# The same in 64 bits, in plain torch: levels, states and hand-derived gradients.
# ---------------------------------------------------------------------------

def _exact_levels(child):
    level = np.zeros(child.shape[0], dtype=np.int64)
    for v, row in enumerate(child.tolist()):        # ids are topological: children first
        kids = [level[c] for c in row if c >= 0]
        level[v] = 1 + max(kids) if kids else 0
    return level


def _exact_schedule(wl):
    child = wl.child
    V = child.shape[0]
    level = _exact_levels(child)
    order = np.argsort(level, kind="stable")
    pos = np.empty(V, dtype=np.int64)
    pos[order] = np.arange(V)
    to_pos = lambda a: np.where(a >= 0, pos[np.maximum(a, 0)], -1)
    offs = np.concatenate([[0], np.cumsum(np.bincount(level))])
    pull, push = wl.pull_idx[order], wl.push_idx[order]
    out = dict(level=level, order=order, pos=pos, child_pos=to_pos(child[order]).reshape(-1),
               parent_pos=to_pos(wl.parent[order]), pull_pos=pull, push_pos=push,
               level_offsets=offs, pull_list=np.nonzero(pull >= 0)[0])
    return {k: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)) for k, a in out.items()}


def exact(case, seed):
    wl = _workload(case, seed)
    if case["kind"] == "schedule":
        return _exact_schedule(wl)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    f64 = lambda a: torch.from_numpy(np.asarray(a, dtype=np.float64)).to(dev)
    idx = lambda a: torch.from_numpy(np.asarray(a, dtype=np.int64)).to(dev)
    V, H, N = wl.V, wl.H, wl.N
    lstm = wl.cell == W.CELL_TREE_LSTM
    level = _exact_levels(wl.child)
    by_level = np.argsort(level, kind="stable")
    cuts = np.cumsum(np.bincount(level))[:-1]
    tasks = [idx(t) for t in np.split(by_level, cuts)]
    child, present = idx(np.maximum(wl.child, 0)), idx(wl.child >= 0).to(torch.float64)
    X, U, b = f64(wl.X), f64(wl.U), f64(wl.b)
    pull = idx(wl.pull_idx)
    zeros = lambda *n: torch.zeros(*n, dtype=torch.float64, device=dev)
    h, c = zeros(V, H), zeros(V, H)
    rows = idx(np.nonzero(wl.pull_idx >= 0)[0])
    if lstm:
        P = zeros(V, 4 * H)
        P[rows] = X[pull[rows]] @ f64(wl.Wx)
        P += b
        Ui, Uf, Uo = U[:, :H], U[:, H:2 * H], U[:, 2 * H:]
        gates = zeros(V, 3, H)                              # i, o, u
        F = zeros(V, N, H)
    for t in tasks:
        kids, on = child[t], present[t].unsqueeze(2)
        hk = h[kids] * on
        if not lstm:
            leaf = (present[t].sum(1) == 0).unsqueeze(1)
            z = torch.tanh(hk.reshape(len(t), N * H) @ U + b)
            x = zeros(len(t), H)
            has = pull[t] >= 0
            x[has] = X[pull[t][has]]
            h[t] = torch.where(leaf, x, z)
            continue
        hs = hk.sum(1)
        p = P[t]
        i = torch.sigmoid(p[:, :H] + hs @ Ui)
        ou = p[:, 2 * H:] + hs @ Uo
        o, u = torch.sigmoid(ou[:, :H]), torch.tanh(ou[:, H:])
        f = torch.sigmoid(p[:, None, H:2 * H] + hk @ Uf) * on
        ct = i * u + (f * c[kids]).sum(1)
        c[t], h[t] = ct, o * torch.tanh(ct)
        gates[t] = torch.stack([i, o, u], 1)
        F[t] = f
    # the head: mean over labelled vertices
    lab = idx(np.nonzero(wl.push_idx >= 0)[0])
    tgt = idx(wl.push_idx)[lab]
    n_lab = max(1, len(lab))
    dh, dc = zeros(V, H), zeros(V, H)
    out = {}
    if wl.loss == W.LOSS_CE:
        Ws = f64(wl.Ws)
        z = h[lab] @ Ws + f64(wl.bs)
        lse = torch.logsumexp(z, 1)
        loss = (lse - z.gather(1, tgt[:, None])[:, 0]).sum() / n_lab
        dz = torch.exp(z - lse[:, None])
        dz[torch.arange(len(lab), device=dev), tgt] -= 1.0
        dz /= n_lab
        dh[lab] = dz @ Ws.t()
        out["dWs"], out["dbs"] = h[lab].t() @ dz, dz.sum(0)
    else:
        d = h[lab] - f64(wl.Y)[tgt]
        loss = 0.5 * (d * d).sum() / n_lab
        dh[lab] = d / n_lab
    res = {"h": h, "loss": loss.reshape(1)}
    if lstm:
        res["c"] = c
    if case["kind"] == "infer":
        return res
    dX = zeros(wl.n_x, wl.D)
    dU = torch.zeros_like(U)
    if lstm:
        dA = zeros(V, 4 * H)                                # i | sum of f_k | o | u
        for t in reversed(tasks):
            kids, on = child[t], present[t].unsqueeze(2)
            i, o, u = gates[t].unbind(1)
            f, ck = F[t], c[kids]
            th = torch.tanh(c[t])
            dct = dc[t] + dh[t] * o * (1 - th * th)
            ai, ao, au = dct * u * i * (1 - i), dh[t] * th * o * (1 - o), dct * i * (1 - u * u)
            af = dct[:, None] * ck * f * (1 - f) * on
            dA[t] = torch.cat([ai, af.sum(1), ao, au], 1)
            hk = h[kids] * on
            hs = hk.sum(1)
            dU[:, :H] += hs.t() @ ai
            dU[:, 2 * H:] += hs.t() @ torch.cat([ao, au], 1)
            dU[:, H:2 * H] += hk.reshape(-1, H).t() @ af.reshape(-1, H)
            dhs = ai @ Ui.t() + torch.cat([ao, au], 1) @ Uo.t()
            dhk = (dhs[:, None] + af @ Uf.t()) * on
            dh.index_add_(0, kids.reshape(-1), dhk.reshape(-1, H))
            dc.index_add_(0, kids.reshape(-1), (dct[:, None] * f).reshape(-1, H))
        out["dWx"] = X[pull[rows]].t() @ dA[rows]
        dX[pull[rows]] = dA[rows] @ f64(wl.Wx).t()
        out["db"] = dA.sum(0)
    else:
        db = torch.zeros_like(b)
        for t in reversed(tasks[1:]):
            kids, on = child[t], present[t].unsqueeze(2)
            a = dh[t] * (1 - h[t] * h[t])
            hk = (h[kids] * on).reshape(len(t), N * H)
            dU += hk.t() @ a
            db += a.sum(0)
            dhk = (a @ U.t()).reshape(len(t), N, H) * on
            dh.index_add_(0, kids.reshape(-1), dhk.reshape(-1, H))
        dX[pull[rows]] = dh[rows]
        out["db"] = db
    res.update(out, dU=dU, dX=dX)
    return res
