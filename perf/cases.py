"""The work that programs hand to this library, as cases that can be timed.

A case is a dict of plain values; prepare() makes what a program holds before
the call (the graph in device memory, a workspace, a plan, the network), run()
makes one pass through the public entry points of paper_1212_4779_amd, work()
says what a pass cannot do without.

Kinds:
  select      StaticGreedy with the dynamic update (select), with the trace of
              every round's gains where the program collects training samples
  lazy        lazy exact evaluation (select_lazy), in bound order or with the
              trained network sizing the batches
  plan        a replay of the selection captured as one graph (Plan)
  batch       several uneven instances selected together (select_batch)
  lt          select on linear-threshold snapshots
  undirected  the component method (select_undirected), one coin per pair
  spread      scoring a seed sequence on independent snapshots (spread)
  mlp         the scoring network: forward, loss and gradient

Graphs are power-law graphs of the shapes that graphgen.WORKLOADS and
graphgen.batch_instances use (weights (i+1)^(-1/(gamma-1)), independent
permutations for out- and in-weights on directed graphs), drawn on the GPU
from the seed, so every seed gives another graph. p = 0 stands for weighted
cascade, p(u,v) = 1/indeg(v).
"""
import math

import numpy as np
import torch

import paper_1212_4779_amd as im
from paper_1212_4779_amd import train_mlp

DEV = "cuda:0"


def _case(kind, n, deg, p, R, k, gamma=2.5, directed=True, **more):
    m = int(n * deg)
    c = dict(kind=kind, n=n, m=m if directed else m - m % 2, gamma=gamma, directed=directed, p=p,
             R=R, k=k)
    c.update(more)
    return c


def listed():
    def named(name, c):
        return dict(c, name=name)

    return [
        # the smallest call: the repository's tiny_uic workload (2,000 nodes)
        named("select_tiny_uic", dict(_case("select", 2000, 10, 0.05, 64, 10), m=20000)),
        # the paper's NetHEPT setting: undirected weighted cascade, ragged R
        named("select_nethept_wc", dict(_case("select", 15000, 4, 0.0, 100, 50, directed=False),
                                        m=59000)),
        # a training graph of the network: weighted cascade, every round's
        # gain vector kept (an odd size)
        named("select_trace_wc_60k", _case("select", 60013, 9.7, 0.0, 128, 20, trace=True)),
        # the headline workload: 10^6 nodes, 10^7 arcs, p = 0.01, R = 256
        named("select_million_uic", _case("select", 1000000, 10, 0.01, 256, 50, gamma=2.1)),
        # the same selection by lazy exact evaluation, four candidates a batch
        named("lazy_million_uic", _case("lazy", 1000000, 10, 0.01, 256, 50, gamma=2.1, batch=4,
                                        learned=False)),
        # a small graph served again and again by one captured plan
        named("plan_uic_20k", _case("plan", 20011, 8.3, 0.05, 130, 20)),
        # uneven instances together: the batched workload's recipe
        named("batch_16", dict(kind="batch", count=16, lo=1000, hi=20000, k=20)),
        # linear threshold at NetHEPT's shape and on a larger directed graph
        named("lt_nethept", dict(_case("lt", 15000, 4, 0.0, 100, 50, directed=False), m=59000)),
        named("lt_200k", _case("lt", 200000, 10, 0.0, 256, 50, gamma=2.1)),
        # undirected graphs at a DBLP-like scale
        named("undirected_million", _case("undirected", 1000000, 10, 0.01, 256, 50, gamma=2.1,
                                          directed=False)),
        # scoring 50 seeds on 20,000 independent snapshots (the accuracy study)
        named("spread_nethept", dict(_case("spread", 15000, 4, 0.0, 20000, 50, directed=False),
                                     m=59000)),
        # one minibatch of the network's training, and its scores
        named("mlp_1024", dict(kind="mlp", samples=1024)),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["select", "select", "lazy", "plan", "batch", "lt", "undirected", "spread",
                       "mlp"])
    if kind == "mlp":
        return dict(kind=kind, samples=_log_int(rng, 1, 200000))
    if kind == "batch":
        return dict(kind=kind, count=rng.randint(2, 16), lo=_log_int(rng, 500, 2000),
                    hi=_log_int(rng, 4000, 20000), k=rng.randint(3, 20))
    gamma = round(rng.uniform(2.1, 2.5), 3)
    deg = round(rng.uniform(4.0, 12.0), 3)
    R = rng.choice([rng.randint(1, 256), 64, 100, 128, 200, 256])
    k = rng.randint(3, 50)
    if kind == "spread":
        n, p = _log_int(rng, 2000, 60000), rng.choice([0.0, 0.01, 0.05])
        return _case(kind, n, deg, p, min(_log_int(rng, 100, 20000), 300000000 // n), k, gamma,
                     p == 0.05 or rng.random() < 0.5)
    if kind == "undirected":
        return _case(kind, _log_int(rng, 2000, 1000000), deg, rng.choice([0.01, 0.02]), R, k, gamma,
                     False)
    if kind == "lt":
        return _case(kind, _log_int(rng, 2000, 150000), deg, 0.0, R, k, gamma, rng.random() < 0.7)
    # weighted cascade is near-critical: its reach sets are far larger
    p = rng.choice([0.0, 0.01, 0.05])
    n = _log_int(rng, 1000, {0.0: 30000, 0.01: 600000, 0.05: 60000}[p])
    directed = True
    if p == 0.0:
        R, k, directed = min(R, 130), min(k, 30), rng.random() < 0.5
    more = {}
    if kind == "select":
        more = dict(trace=rng.random() < 0.3)
    elif kind == "lazy":
        more = dict(batch=rng.choice([1, 4, 16]), learned=rng.random() < 0.5)
    return _case(kind, n, deg, p, R, k, gamma, directed, **more)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _arcs(n, m, gamma, directed, g):
    """Sorted keys tail * n + head of m distinct arcs (or of m / 2 pairs, both directions)."""
    target = m if directed else m // 2
    cdf = np.cumsum((np.arange(n, dtype=np.float64) + 1.0) ** (-1.0 / (gamma - 1.0)))
    cdf = torch.from_numpy(cdf / cdf[-1]).to(DEV)
    out = torch.randperm(n, generator=g, device=DEV)
    inn = torch.randperm(n, generator=g, device=DEV) if directed else out
    keys = torch.empty(0, dtype=torch.int64, device=DEV)
    while keys.numel() < target:
        b = int((target - keys.numel()) * 1.3) + 1024
        u = torch.rand((2, b), generator=g, device=DEV, dtype=torch.float64)
        a = out[torch.searchsorted(cdf, u[0], right=True).clamp_(max=n - 1)]
        c = inn[torch.searchsorted(cdf, u[1], right=True).clamp_(max=n - 1)]
        if not directed:
            a, c = torch.minimum(a, c), torch.maximum(a, c)
        keys = torch.unique(torch.cat([keys, (a * n + c)[a != c]]))
    pick = torch.randperm(keys.numel(), generator=g, device=DEV)[:target]
    keys = keys[pick]
    if not directed:
        keys = torch.cat([keys, (keys % n) * n + keys // n])
    return torch.sort(keys).values


def _graph(n, m, gamma, directed, p, g):
    keys = _arcs(n, m, gamma, directed, g)
    src, dst = keys // n, keys % n
    row = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(torch.bincount(src, minlength=n), 0, out=row[1:])
    if p:
        prob = torch.full((m,), p, dtype=torch.float32, device=DEV)
    else:
        prob = 1.0 / torch.bincount(dst, minlength=n).to(torch.float32)[dst]
    return im.Graph(row, dst.to(torch.int32), prob)


def _batch(case):
    """(n, m, p, R) of every instance: a fixed uneven mix of the case's range."""
    rng = np.random.default_rng(case["count"] * 1000003 + case["hi"])
    out = []
    for i in range(case["count"]):
        n = int(round(math.exp(rng.uniform(math.log(case["lo"]), math.log(case["hi"])))))
        p = (0.01 if (i // 2) % 2 == 0 else 0.05) if i % 2 == 0 else 0.0
        out.append((n, int(round(n * rng.uniform(4.0, 16.0))), p, int(rng.choice([64, 128, 256]))))
    return out


def _samples(case, g):
    """Network inputs as node features are (logarithms of degrees and gains) and targets below
    the last gain, as later gains are."""
    n = case["samples"]
    x = torch.log1p(torch.empty((n, im.api.MLP_IN), device=DEV).exponential_(0.1, generator=g))
    t = x[:, 4] * torch.rand(n, generator=g, device=DEV)
    return x, t


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    if kind == "mlp":
        x, t = _samples(case, g)
        return dict(case=case, net=train_mlp.load(), x=x, t=t)
    if kind == "batch":
        inst = [(_graph(n, m, 2.5, True, p, g), R, case["k"], int(seed) + i)
                for i, (n, m, p, R) in enumerate(_batch(case))]
        return dict(case=case, instances=inst, ws=im.Workspace())
    graph = _graph(case["n"], case["m"], case["gamma"], case["directed"], case["p"], g)
    s = dict(case=case, graph=graph, seed=int(seed) + 1)
    if kind == "plan":
        s["plan"] = im.Plan(graph, case["R"], case["k"], s["seed"])
        return s
    s["ws"] = im.Workspace()
    if kind == "lt":
        s["ws"].set_live_edge(1)
    if kind == "spread":
        # the seeds of a selection lean to nodes of many arcs
        deg = graph.row_ptr[1:] - graph.row_ptr[:-1]
        top = torch.topk(deg, min(case["n"], 4 * case["k"])).indices
        s["seeds"] = top[torch.randperm(top.numel(), generator=g, device=DEV)[:case["k"]]]
    if kind == "lazy":
        s["net"] = train_mlp.load() if case["learned"] else None
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "select" or kind == "lt":
        seeds, gains, trace = im.select(s["graph"], case["R"], case["k"], s["seed"], ws=s["ws"],
                                        trace=bool(case.get("trace")))
        return dict(seeds=seeds, gains=gains, trace=trace)
    if kind == "lazy":
        seeds, gains = im.select_lazy(s["graph"], case["R"], case["k"], s["seed"],
                                      batch=case["batch"], model=s["net"], ws=s["ws"])
        return dict(seeds=seeds, gains=gains)
    if kind == "plan":
        s["plan"].launch()
        return dict(seeds=s["plan"].seeds, gains=s["plan"].gains)
    if kind == "batch":
        return [list(r) for r in im.select_batch(s["instances"], ws=s["ws"])]
    if kind == "undirected":
        seeds, gains, _ = im.select_undirected(s["graph"], case["R"], case["k"], s["seed"],
                                               ws=s["ws"])
        return dict(seeds=seeds, gains=gains)
    if kind == "spread":
        marg, per = im.spread(s["graph"], case["R"], s["seed"], s["seeds"], ws=s["ws"],
                              per_snapshot=True)
        return dict(marg=marg, per=per)
    loss, grad = s["net"].loss_grad(s["x"], s["t"])
    return dict(y=s["net"].forward(s["x"]), loss=loss, grad=grad)


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
DRAW_OPS = 22   # integer operations of one coin (two SplitMix64 mixes, a comparison)


def _graph_bytes(n, m):
    return 8 * (n + 1) + 8 * m   # row offsets, heads and probabilities


def work(case):
    kind = case["kind"]
    if kind == "mlp":
        n = case["samples"]
        mac = im.api.MLP_IN * 64 + 64 * 64 + 64   # per sample, forward; the gradient takes twice
        return dict(bytes=4 * n * (im.api.MLP_IN + 2) + 2 * 4 * im.api.MLP_NPARAM, flops=6 * n * mac)
    if kind == "batch":
        inst = _batch(case)
        return dict(bytes=sum(_graph_bytes(n, m) for n, m, _, _ in inst) + 12 * case["k"] * len(inst),
                    flops=sum(DRAW_OPS * m * R for _, m, _, R in inst))
    n, m, R, k = case["n"], case["m"], case["R"], case["k"]
    out = 12 * k + (4 * (k + 1) * n if case.get("trace") else 0)
    if kind == "lt":         # one draw per (node, snapshot)
        return dict(bytes=_graph_bytes(n, m) + out, flops=DRAW_OPS * n * R)
    if kind == "undirected":   # one coin per pair
        return dict(bytes=_graph_bytes(n, m) + out, flops=DRAW_OPS * (m // 2) * R)
    if kind == "spread":     # at least the seeds' own arcs
        return dict(bytes=_graph_bytes(n, m) + 8 * k + 4 * R, flops=DRAW_OPS * (m // n + 1) * k * R)
    return dict(bytes=_graph_bytes(n, m) + out, flops=DRAW_OPS * m * R)


def exact(case, seed):
    """The network's outputs in 64 bits. Every other kind returns whole numbers (seeds, counts),
    which have to stay equal, so there is nothing to be nearer to."""
    if case["kind"] != "mlp":
        return None
    x, t = (v.double() for v in _samples(case, _gen(seed)))
    net = train_mlp.load()
    bits = net.params()[1]   # the network computes with its bfloat16 weights
    net.close()
    p = torch.from_numpy((bits.astype(np.uint32) << 16).view(np.float32).astype(np.float64)).to(DEV)
    p.requires_grad_(True)
    h = im.api.MLP_IN
    w1, b1, w2, b2, w3, b3 = torch.split(p, [64 * h, 64, 64 * 64, 64, 64, 1])
    a1 = torch.relu(x @ w1.view(64, h).t() + b1)
    a2 = torch.relu(a1 @ w2.view(64, 64).t() + b2)
    y = a2 @ w3 + b3
    loss = (y - t).square().sum() / (2 * x.shape[0])
    (grad,) = torch.autograd.grad(loss, p)
    return dict(y=y.detach(), loss=loss.detach().reshape(1), grad=grad)
