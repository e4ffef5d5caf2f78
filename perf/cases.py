"""Performance cases: the work a program has this library do, as calls of the
public entry points in ``paper_2507_14813_amd.api``.

Every case is a dict of plain values.  ``kind`` names the call:

* ``count``      one ``api.count`` over a resident graph (co-mining, or one
                 search per motif with ``mode``), one window or several
* ``serve``      ``api.count_noalloc``: a serving loop that allocates nothing
* ``batch``      ``api.Batch.count``: many jobs replayed as one launch; with
                 ``oneshot`` ``api.count_batch`` (planned and counted once)
* ``enumerate``  ``api.enumerate_matches``, in a fixed order
* ``load``       ``api.Graph`` from unsorted device arrays, then one count
* ``learned``    ``api.count`` with the learned root-cost schedule
* ``fit``        ``api.root_features``, ``Model.train``, ``Model.predict``

Graphs are seeded and drawn on the GPU with integer prefix sums, so that one
seed always gives the same graph.  The recipe is that of
``workloads.powerlaw_graph`` / ``uniform_graph``: heavy-tailed directed degrees
capped at sqrt(E), per-source Pareto bursts with 30 s gaps, destinations
repeated inside a burst with probability 0.5.
"""
import math

import numpy as np
import torch

from paper_2507_14813_amd import api
from paper_2507_14813_amd import workloads as W

DEV = "cuda"
SPAN = 30_000_000          # seconds, about a year


# --------------------------------------------------------------------- cases
def _case(name=None, kind="count", graph="powerlaw", edges=20_000, nodes=2_000, gamma=2.1,
          span=SPAN, burst_cap=0, ns=False, motifs="triads", n_motifs=0, mseed=0, delta=3600,
          windows=1, mode="comine", jobs=0, smallest=0, oneshot=False, rows=0, epochs=0):
    c = dict(kind=kind, graph=graph, edges=edges, nodes=nodes, gamma=gamma, span=span,
             burst_cap=burst_cap, ns=ns, motifs=motifs, n_motifs=n_motifs, mseed=mseed,
             delta=delta, windows=windows, mode=mode, jobs=jobs, smallest=smallest,
             oneshot=oneshot, rows=rows, epochs=epochs)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one request of a serving loop on a tiny graph: launch latency
        _case("serve_1k", "serve", "uniform", 1_000, 100, span=50_000, motifs="path",
              delta=10_000),
        # the small uniform workload: 2,000 nodes, 20,000 edges, four path motifs
        _case("uniform_20k", "count", "uniform", 20_000, 2_000, span=1_000_000, motifs="path",
              delta=10_000),
        # the 36 three-edge motifs on a graph of ordinary size, odd edge count
        _case("triads_2m", edges=2_000_003, nodes=100_000),
        # the benchmark workload: 20M edges, 36 motifs, one-hour window
        _case("triads_20m", edges=20_000_000, nodes=1_000_000),
        # all 756 three- and four-edge motifs on <= 4 nodes, steeper degrees, 2 h
        _case("quads_3m", edges=3_000_000, nodes=300_000, gamma=1.8, burst_cap=64,
              motifs="quads", delta=7200),
        # a window sweep: 48 motifs of 3-5 edges, three windows in one search
        _case("sweep_4m", edges=4_000_001, nodes=400_000, gamma=2.0, span=100_000_000,
              burst_cap=32, motifs="walks", n_motifs=48, mseed=51, delta=21600, windows=3),
        # one search per motif (the comparison mode) on nanosecond times (64 bit)
        _case("per_motif_ns_1m", edges=1_000_000, nodes=50_000, ns=True, mode="per_motif"),
        # a plan of 24 uneven jobs replayed as one launch
        _case("batch_24", "batch", edges=250_000, nodes=0, smallest=10_000, jobs=24,
              burst_cap=64, motifs="mixed", mseed=3000),
        # every match written out: three-edge motifs on a 200k-edge graph
        _case("enumerate_200k", "enumerate", edges=200_000, nodes=10_000, burst_cap=64),
        # a new graph, unsorted, in device memory: loaded and counted once
        _case("load_1m", "load", edges=1_000_003, nodes=50_000),
        # the learned schedule on a mid-size graph
        _case("learned_2m", "learned", edges=2_000_000, nodes=100_000),
        # the cost model: features of sampled roots, training, prediction
        _case("fit_16k", "fit", edges=500_000, nodes=25_000, rows=16_384, epochs=2),
    ]


def _loguniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["count"] * 8 + ["serve", "batch", "batch", "enumerate", "load", "load",
                                       "learned", "fit"])
    gamma = round(rng.uniform(1.8, 2.5), 3)
    delta = rng.choice([600, 900, 3600, 7200])
    if kind == "serve" or (kind == "count" and rng.random() < 0.25):
        e = _loguniform(rng, 1_000, 60_000)
        n = max(16, e // rng.choice([5, 10, 20]))
        return _case(None, kind, "uniform", e, n, span=50 * e, ns=rng.random() < 0.2,
                     motifs=rng.choice(["path", "triads"]), delta=rng.choice([2_000, 10_000]))
    if kind == "count":
        motifs = rng.choice(["triads", "triads", "quads", "walks"])
        top = {"triads": 8_000_000, "quads": 2_000_000, "walks": 3_000_000}[motifs]
        mode = "comine" if motifs == "quads" or rng.random() < 0.8 else "per_motif"
        e = _loguniform(rng, 60_000, top if mode == "comine" else 1_000_000)
        return _case(None, kind, edges=e, nodes=e // rng.choice([10, 20]), gamma=gamma,
                     burst_cap=rng.choice([0, 64]) if motifs == "triads" else 32,
                     ns=rng.random() < 0.25, motifs=motifs,
                     n_motifs=rng.randint(8, 48) if motifs == "walks" else 0,
                     mseed=rng.randint(0, 999), delta=delta,
                     windows=rng.choice([1, 1, 3]), mode=mode)
    if kind == "batch":
        return _case(None, kind, edges=_loguniform(rng, 40_000, 250_000), nodes=0,
                     smallest=rng.choice([1_000, 10_000]), jobs=rng.randint(2, 24),
                     burst_cap=64, gamma=gamma, motifs="mixed", mseed=rng.randint(0, 9999),
                     ns=rng.random() < 0.2, oneshot=rng.random() < 0.4)
    if kind == "enumerate":
        e = _loguniform(rng, 20_000, 250_000)
        return _case(None, kind, edges=e, nodes=e // 20, gamma=gamma, burst_cap=32,
                     mseed=rng.randint(0, 999), delta=rng.choice([600, 3600]))
    if kind == "load":
        e = _loguniform(rng, 20_000, 2_000_000)
        return _case(None, kind, edges=e, nodes=e // rng.choice([10, 20]), gamma=gamma,
                     burst_cap=rng.choice([0, 64]), ns=rng.random() < 0.3, delta=delta)
    if kind == "learned":
        e = _loguniform(rng, 100_000, 3_000_000)
        return _case(None, kind, edges=e, nodes=e // 20, gamma=gamma, burst_cap=64, delta=delta)
    return _case(None, "fit", edges=_loguniform(rng, 50_000, 500_000), nodes=20_000, gamma=gamma,
                 burst_cap=64, delta=delta, rows=32 * rng.randint(64, 512),
                 epochs=rng.randint(1, 2))


# -------------------------------------------------------------------- inputs
def _gen(seed, salt):
    g = torch.Generator(DEV)
    g.manual_seed((int(seed) * 1_000_003 + salt) & 0x7fffffffffff)
    return g


def _times(g, t, ns):
    if not ns:
        return t
    return t * 1_000_000_000 + torch.randint(0, 1_000_000_000, t.shape, generator=g, device=DEV)


def _uniform(g, V, E, span):
    src = torch.randint(0, V, (E,), generator=g, device=DEV)
    dst = (src + torch.randint(1, V, (E,), generator=g, device=DEV)) % V
    return src, dst, torch.randint(0, span, (E,), generator=g, device=DEV)


def _weights(g, V, gamma, cap):
    """Integer prefix sums of Pareto weights (tail gamma - 1, capped)."""
    u = torch.rand(V, generator=g, device=DEV, dtype=torch.float64).clamp_min(1e-12)
    w = (u ** (-1.0 / (gamma - 1.0))).clamp_max(cap)
    return (w * 65536).to(torch.int64).cumsum(0)


def _pick(g, cdf, n):
    top = int(cdf[-1])
    x = torch.randint(0, top, (n,), generator=g, device=DEV)
    return torch.searchsorted(cdf, x, right=True)


def _powerlaw(g, V, E, gamma, span, burst_cap):
    cap = math.sqrt(E)
    out, into = _weights(g, V, gamma, cap), _weights(g, V, gamma, cap)
    into_id = torch.randperm(V, generator=g, device=DEV)
    src = _pick(g, out, E).sort().values                 # grouped by source
    size = torch.rand(E, generator=g, device=DEV, dtype=torch.float64).clamp_min(1e-12)
    size = (size ** (-1.0 / 1.5)).ceil().clamp_max(burst_cap or 1e9).to(torch.int64)
    start = torch.ones(E + 1, dtype=torch.bool, device=DEV)
    start[1:E] = src[1:] != src[:-1]                     # a source starts a burst
    start[size.cumsum(0).clamp_max(E)] = True
    start = start[:E]
    first = start.nonzero().flatten()
    burst = start.cumsum(0) - 1
    begin = torch.randint(0, span, first.shape, generator=g, device=DEV)
    gap = torch.rand(E, generator=g, device=DEV, dtype=torch.float64).clamp_min(1e-12)
    gap = (gap.log() * (-30.0 * 1024)).to(torch.int64)   # exponential, mean 30 s
    gap[start] = 0
    run = gap.cumsum(0)
    t = (begin[burst] + (run - run[first][burst]) // 1024).clamp(0, span - 1)
    dst = into_id[_pick(g, into, E)]
    dst = torch.where(dst == src, (dst + 1) % V, dst)
    again = (torch.rand(E, generator=g, device=DEV) < 0.5) & ~start
    pos = torch.where(again, torch.zeros_like(src), torch.arange(E, device=DEV))
    return src, dst[pos.cummax(0).values], t


def _edges(case, seed, salt=0, edges=None, nodes=None, is_sorted=True):
    """(src int32, dst int32, t int64) on the GPU, in time order or shuffled."""
    g = _gen(seed, salt)
    E = edges or case["edges"]
    V = nodes or case["nodes"]
    if case["graph"] == "uniform":
        s, d, t = _uniform(g, V, E, case["span"])
    else:
        s, d, t = _powerlaw(g, V, E, case["gamma"], case["span"], case["burst_cap"])
    t = _times(g, t, case["ns"])
    o = t.sort(stable=True).indices if is_sorted else torch.randperm(E, generator=g, device=DEV)
    return s[o].to(torch.int32), d[o].to(torch.int32), t[o].contiguous()


def _relabelled(case, seed):
    """One graph per case under the seed's vertex names and edge order, so
    that every seed has as many matches (and other records)."""
    s, d, t = _edges(case, case["mseed"])
    g = _gen(seed, 5)
    name = torch.randperm(case["nodes"], generator=g, device=DEV).to(torch.int32)
    o = torch.randperm(case["edges"], generator=g, device=DEV)
    return name[s[o].long()], name[d[o].long()], t[o]


def _unit(case):
    return 1_000_000_000 if case["ns"] else 1


def _deltas(case):
    d = case["delta"] * _unit(case)
    return [d // 24, d // 6, d] if case["windows"] == 3 else d


def _motifs(case):
    m = case["motifs"]
    if m == "path":
        return list(W.CONFIG1_MOTIFS)
    if m == "triads":
        return W.enumerate_motifs(3, 3)
    if m == "quads":
        return W.enumerate_motifs(3, 4) + W.enumerate_motifs(4, 4)
    n, s = case["n_motifs"], case["mseed"]
    parts = [n - 2 * (n // 3), n // 3, n // 3]
    return [x for k, p in zip((3, 4, 5), parts)
            for x in W.random_extension_motifs(p, (k,), 5, s + k)]


def _batch_jobs(case):
    """Per job: edges, nodes, motif set, window (fixed by the case)."""
    rng = np.random.Generator(np.random.PCG64(case["mseed"]))
    jobs = []
    for j in range(case["jobs"]):
        e = int(round(math.exp(rng.uniform(math.log(case["smallest"]), math.log(case["edges"])))))
        nm = int(rng.integers(4, 25))
        jobs.append((e, max(16, e // 10),
                     W.random_extension_motifs(nm, (2, 3, 4), 5, case["mseed"] + j),
                     int(rng.choice([600, 3600, 86400])) * _unit(case)))
    return jobs


def _graph(case, seed):
    return api.Graph(*_edges(case, seed), n_nodes=case["nodes"], sorted_by_t=True)


def _sampled_roots(case, seed):
    rng = np.random.Generator(np.random.PCG64(int(seed) + 17))
    return np.sort(rng.integers(0, case["edges"], case["rows"] or 8192))


def _start_weights(seed):
    rng = np.random.Generator(np.random.PCG64(int(seed) + 29))
    w = np.zeros(api.MODEL_PARAMS, np.float32)
    for off, fan, n in ((0, 16, 16 * 64), (2112, 64, 4096), (6272, 64, 4096), (10432, 64, 64)):
        w[off:off + n] = rng.standard_normal(n) * math.sqrt(2.0 / fan)
    return w


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        jobs = _batch_jobs(case)
        graphs = [api.Graph(*_edges(case, seed, j + 1, e, v), n_nodes=v, sorted_by_t=True)
                  for j, (e, v, _, _) in enumerate(jobs)]
        trees = [api.Tree(m, d) for _, _, m, d in jobs]
        if case["oneshot"]:
            return {"kind": "oneshot", "graphs": graphs, "trees": trees}
        return {"kind": kind, "batch": api.Batch(graphs, trees)}
    tree = api.Tree(_motifs(case), _deltas(case))
    if kind == "load":
        return {"kind": kind, "tree": tree, "nodes": case["nodes"],
                "edges": _edges(case, seed, is_sorted=False)}
    if kind == "enumerate":
        return {"kind": kind, "tree": tree,
                "graph": api.Graph(*_relabelled(case, seed), n_nodes=case["nodes"])}
    st = {"kind": kind, "graph": _graph(case, seed), "tree": tree, "mode": case["mode"]}
    if kind == "serve":
        api.count(st["graph"], tree)          # puts the tree's tables on the device
    if kind in ("learned", "fit"):
        roots = _sampled_roots(case, seed)
        _, cost = api.count(st["graph"], tree, roots=roots, root_cost=True)
        labels = np.log1p(cost[roots].astype(np.float64)).astype(np.float32)
        st.update(roots=roots, labels=labels, start=_start_weights(seed), epochs=case["epochs"])
        st["model"] = api.Model(weights=st["start"])
        if kind == "learned":
            st["model"].train(api.root_features(st["graph"], tree, roots), labels, 1, 1e-3, seed=1)
    return st


# ----------------------------------------------------------------- one pass
def run(st):
    kind = st["kind"]
    if kind == "count":
        return api.count(st["graph"], st["tree"], mode=st["mode"])
    if kind == "serve":
        return api.count_noalloc(st["graph"], st["tree"])
    if kind == "batch":
        return np.concatenate([c.reshape(-1) for c in st["batch"].count()])
    if kind == "oneshot":
        parts = api.count_batch(st["graphs"], st["trees"])
        return np.concatenate([c.reshape(-1) for c in parts])
    if kind == "enumerate":
        motif, edges = api.enumerate_matches(st["graph"], st["tree"])
        # records come in no particular order; three edges of under 2^18 and a
        # motif index order them in one 64-bit key, which holds the whole record
        key = motif.astype(np.int64)
        for k in range(3):
            key = (key << 18) | edges[:, k]
        key.sort()
        return key
    if kind == "load":
        g = api.Graph(*st["edges"], n_nodes=st["nodes"])
        return api.count(g, st["tree"])
    if kind == "learned":
        return api.count(st["graph"], st["tree"], model=st["model"])
    m = st["model"]
    m.set_weights(st["start"])
    feats = api.root_features(st["graph"], st["tree"], st["roots"])
    loss = m.train(feats, st["labels"], st["epochs"], 1e-3, seed=1)
    return {"features": feats, "loss": loss, "weights": m.weights(), "pred": m.predict(feats)}


def work(case):
    """Bytes: the edges (two ids and a time each) read once, the results
    written once.  What a search has to examine beyond that depends on the
    graph, so it is left out.  Operations: the cost model's products."""
    tb = 8 if case["ns"] else 4
    kind = case["kind"]
    if kind == "batch":
        jobs = _batch_jobs(case)
        return {"bytes": sum(e * (8 + tb) + 8 * len(m) for e, _, m, _ in jobs), "flops": 0}
    if kind == "fit":
        n, macs = case["rows"], 16 * 64 + 2 * 64 * 64 + 64
        steps = n * case["epochs"]
        return {"bytes": n * (8 + 4 + 4 * 16 + 4) + 3 * 4 * api.MODEL_PARAMS,
                "flops": 2 * macs * (3 * steps + n)}
    n_out = len(_motifs(case)) * case["windows"]
    if kind == "load":
        return {"bytes": case["edges"] * 16 + 8 * n_out, "flops": 0}
    return {"bytes": case["edges"] * (8 + tb) + 8 * n_out, "flops": 0}


# --------------------------------------------------------- 64-bit references
def _count_exact(s, d, t, motifs, delta):
    """Depth-first matching in plain Python (small graphs only)."""
    out = {}
    for i in range(len(s)):
        out.setdefault(s[i], []).append(i)
    total = []
    for m in motifs:
        n = 0
        for r in range(len(s)):
            stack = [((s[r], d[r]), 1, r)] if s[r] != d[r] else []
            while stack:
                phi, k, last = stack.pop()
                if k == len(m):
                    n += 1
                    continue
                u, v = m[k]
                for e in out.get(phi[u], ()):       # every path motif extends a bound source
                    if e <= last or t[e] <= t[last] or t[e] > t[r] + delta:
                        continue
                    x = d[e]
                    if v < len(phi):
                        if x == phi[v]:
                            stack.append((phi, k + 1, e))
                    elif x not in phi:
                        stack.append((phi + (x,), k + 1, e))
        total.append(n)
    return np.array(total, dtype=np.uint64)


def _features_exact(s, d, t, V, tree_depth, n_motifs, delta, roots):
    o, i = np.lexsort((t, s)), np.lexsort((t, d))
    lists = []
    for v, order in ((s, o), (d, i)):
        off = np.concatenate([[0], np.cumsum(np.bincount(v, minlength=V))])
        lists.append((off, t[order]))
    f = np.zeros((len(roots), 16))
    for r, e in enumerate(roots):
        lo, hi, k = t[e], t[e] + delta, 0
        for (off, tt), v, col in ((lists[0], s[e], 0), (lists[1], s[e], 1), (lists[0], d[e], 2),
                                  (lists[1], d[e], 3)):
            seg = tt[off[v]:off[v + 1]]
            f[r, col] = np.log1p(len(seg)) / 16
            k = np.searchsorted(seg, hi, "right") - np.searchsorted(seg, lo, "right")
            f[r, {0: 4, 2: 5, 1: 6, 3: 7}[col]] = np.log1p(k) / 16
        k = np.searchsorted(t, hi, "right") - np.searchsorted(t, lo, "right")
        f[r, 8] = np.log1p(k) / 16
    f[:, 9], f[:, 10], f[:, 11] = tree_depth * 0.125, np.log1p(n_motifs) * 0.125, 1.0
    return f


def _shuffled(n, seed):
    """The documented seeded order of the training rows (splitmix64 shuffle)."""
    mask, s, p = (1 << 64) - 1, int(seed), list(range(n))
    for i in range(n - 1, 0, -1):
        s = (s + 0x9e3779b97f4a7c15) & mask
        z = ((s ^ (s >> 30)) * 0xbf58476d1ce4e5b9) & mask
        z = ((z ^ (z >> 27)) * 0x94d049bb133111eb) & mask
        j = (z ^ (z >> 31)) % (i + 1)
        p[i], p[j] = p[j], p[i]
    return np.array(p)


def _split(w):
    return [w[0:1024].reshape(16, 64), w[2048:2112], w[2112:6208].reshape(64, 64), w[6208:6272],
            w[6272:10368].reshape(64, 64), w[10368:10432], w[10432:10496], w[10496:10497]]


def _forward(p, x):
    h = [x]
    for k in (0, 2, 4):
        h.append(np.maximum(h[-1] @ p[k] + p[k + 1], 0))
    return h, h[-1] @ p[6] + p[7]


def _fit_exact(feats, labels, w, epochs, lr, seed):
    w = w.astype(np.float64)
    m, v, step, loss = np.zeros_like(w), np.zeros_like(w), 0, []
    order = _shuffled(len(feats), seed)
    for _ in range(epochs):
        total, nb = 0.0, len(feats) // 32
        for b in range(nb):
            rows = order[32 * b:32 * b + 32]
            p, g = _split(w), np.zeros_like(w)
            h, out = _forward(p, feats[rows])
            e = out - labels[rows]
            total += float((e * e).sum())
            do = 2 * e / 32
            gp = _split(g)
            gp[6][:], gp[7][:] = h[3].T @ do, do.sum()
            dz = np.outer(do, p[6]) * (h[3] > 0)
            for k, a in ((4, 2), (2, 1), (0, 0)):
                gp[k][:], gp[k + 1][:] = h[a].T @ dz, dz.sum(0)
                if a:
                    dz = (dz @ p[k].T) * (h[a] > 0)
            step += 1
            m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
            w = w - lr * (m / (1 - 0.9 ** step)) / (np.sqrt(v / (1 - 0.999 ** step)) + 1e-8)
        loss.append(total / (nb * 32))
    return np.array(loss), w


def exact(case, seed):
    """Counts are whole numbers, given for the small path cases; the cost
    model's outputs in 64-bit floating point."""
    if case["kind"] == "fit":
        s, d, t = (x.cpu().numpy().astype(np.int64) for x in _edges(case, seed))
        roots = _sampled_roots(case, seed)
        motifs = _motifs(case)
        feats = _features_exact(s, d, t, case["nodes"], max(len(m) for m in motifs), len(motifs),
                                _deltas(case), roots)
        st = prepare(case, seed)      # for the labels (whole numbers) and the start weights
        labels, start = st["labels"].astype(np.float64), st["start"]
        loss, w = _fit_exact(feats, labels, start, case["epochs"], 1e-3, 1)
        return {"features": feats, "loss": loss, "weights": w,
                "pred": _forward(_split(w), feats)[1]}
    if case["kind"] in ("count", "serve") and case["motifs"] == "path" and case["edges"] <= 20_000:
        s, d, t = (x.cpu().numpy().tolist() for x in _edges(case, seed))
        return _count_exact(s, d, t, _motifs(case), _deltas(case))
    return None
