"""Leaf windows counted from pairs, and windows skipped because no list entry
lies in them: bursts between few pairs (long runs of one pair and of its
reverse, ties, a pair that only ever runs one way), isolated edges, windows that
end exactly on an edge, unbounded windows.  Whole numbers, equal to the
oracle's."""
import itertools

import numpy as np
import pytest

import oracle
from paper_2507_14813_amd import workloads as W

pytestmark = pytest.mark.gpu

THREE = W.enumerate_motifs(3, 3)
FOUR = W.enumerate_motifs(3, 4)[::3] + W.enumerate_motifs(4, 4)[::9]
MIXED = ([((0, 1), (0, 1)), ((0, 1), (1, 0), (0, 2)), ((0, 1), (2, 3), (3, 1))] +
         W.random_extension_motifs(12, (2, 3, 4, 5), 5, 77))


@pytest.fixture(scope="module")
def api(oracle_mod):
    import torch
    assert torch.cuda.is_available(), "no GPU visible"
    from paper_2507_14813_amd import api
    api.lib()
    return api


def bursts(n_edges, seed, unit):
    rng = np.random.default_rng(seed)
    s, d, t = [], [], []
    while len(s) < n_edges:
        a, b = rng.choice(14, 2, replace=False)
        k = int(rng.choice([1, 1, 2, 5, 40, 150]))
        t0 = int(rng.integers(0, 60 * n_edges))
        for _ in range(k):
            flip = rng.random() < 0.3 and min(a, b) > 2
            s.append(b if flip else a)
            d.append(a if flip else b)
            t.append(t0)
            t0 += int(rng.choice([0, 1, 3, 9]))
            if rng.random() < 0.3:
                b = int(rng.choice([x for x in range(14) if x != a]))
    return (np.array(s[:n_edges], np.int32), np.array(d[:n_edges], np.int32),
            np.array(t[:n_edges], np.int64) * unit)


@pytest.mark.parametrize("unit", [1, 2 ** 33])
@pytest.mark.parametrize("motifs,n_edges", [(THREE, 6000), (FOUR, 2500), (MIXED, 1500)])
def test_burst_counts_equal_oracle(api, motifs, n_edges, unit):
    s, d, t = bursts(n_edges, n_edges + 1, unit)
    g, og = api.Graph(s, d, t, 15), oracle.OracleGraph(s, d, t, 15)
    deltas = [9 * unit, 120 * unit, 31 * unit]
    print("bursts", len(motifs), n_edges, unit, flush=True)
    want = np.array([[og.count(m, x) for m in motifs] for x in deltas], dtype=np.uint64)
    for i, x in enumerate(deltas):
        tr = api.Tree(motifs, x)
        assert np.array_equal(api.count(g, tr), want[i])
        assert np.array_equal(api.count(g, tr, leaf_scan=-1), want[i])
        assert np.array_equal(api.count(g, tr, epoch_idle=1, max_epochs=3), want[i])
    assert np.array_equal(api.count(g, api.Tree(motifs, deltas)), want)
    assert np.array_equal(np.stack(api.count_batch([g] * 3, [api.Tree(motifs, x) for x in deltas])), want)


def test_unbounded_window_and_isolated_edges(api):
    s, d, t = bursts(60, 5, 1)
    # edges that touch no other edge's vertices within any window
    s = np.concatenate([s, np.arange(20, 60, 2)]).astype(np.int32)
    d = np.concatenate([d, np.arange(21, 61, 2)]).astype(np.int32)
    t = np.concatenate([t, np.arange(20) * 7]).astype(np.int64)
    g, og = api.Graph(s, d, t, 61), oracle.OracleGraph(s, d, t, 61)
    for x in (0, 2 ** 63 - 1):
        want = np.array([og.count(m, x) for m in THREE], dtype=np.uint64)
        assert np.array_equal(api.count(g, api.Tree(THREE, x)), want)


@pytest.mark.parametrize("n_edges", [1, 63, 1000, 1023, 9000, 65_536, 65_537])
def test_small_counts_in_one_launch(api, n_edges):
    """Counts small enough for one launch, around the sizes where the chunk
    length and the choice change: mg_count, mg_count_noalloc, several windows,
    from several threads and streams."""
    import threading

    import torch
    rng = np.random.default_rng(n_edges)
    n = max(4, n_edges // 40)
    s = rng.integers(0, n, n_edges).astype(np.int32)
    d = rng.integers(0, n, n_edges).astype(np.int32)
    t = np.sort(rng.integers(0, 20 * n_edges, n_edges)).astype(np.int64)
    g, og = api.Graph(s, d, t, n), oracle.OracleGraph(s, d, t, n)
    motifs = THREE[::5]
    want = np.array([[og.count(m, x) for m in motifs] for x in (40, 400)], dtype=np.uint64)
    tr = api.Tree(motifs, 400)
    assert np.array_equal(api.count(g, tr), want[1])
    assert np.array_equal(api.count(g, tr, chunk=64), want[1])
    assert np.array_equal(api.count_noalloc(g, tr), want[1])
    assert np.array_equal(api.count(g, api.Tree(motifs, [40, 400])), want)
    bad = []

    def work(k):
        g2, tr2 = api.Graph(s, d, t, n), api.Tree(motifs, 400)
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(20):
                if not np.array_equal(api.count(g2, tr2), want[1]):
                    bad.append(k)

    th = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    [x.start() for x in th]
    [x.join() for x in th]
    assert not bad


@pytest.mark.parametrize("k,delta", [(1, 0), (2, 1), (3, 5), (5, 5)])
@pytest.mark.parametrize("n_edges", [1, 63, 64, 65, 129, 1000])
def test_enumeration_writes_every_staged_match(api, n_edges, k, delta):
    """A run of one pair, one edge per time unit: the matches of its k-edge
    repetition are the index combinations that span at most delta.  One motif
    and a few matches per root, so a wave's staged matches end below, at and
    above 64; a capacity below the total reports the total."""
    import ctypes
    t = np.arange(n_edges, dtype=np.int64)
    z = np.zeros(n_edges, np.int32)
    g = api.Graph(z, z + 1, t, 2)
    tree = api.Tree([((0, 1),) * k], delta)
    want = [c for i in range(n_edges)
            for c in ((i,) + r for r in itertools.combinations(range(i + 1, min(n_edges, i + delta + 1)), k - 1))]
    motif, edges = api.enumerate_matches(g, tree)
    assert (motif == 0).all() and (edges[:, k:] == -1).all()
    assert sorted(map(tuple, edges[:, :k].tolist())) == want
    if len(want) > 1:
        n = ctypes.c_int64(0)
        rec = np.full((len(want) - 1, 6), -7, np.int32)
        assert api.lib().mg_enumerate(g.handle, tree.handle, None, rec.ctypes.data, len(want) - 1,
                                      ctypes.byref(n)) == 0
        assert n.value == len(want) and (rec == -7).all()


def test_one_tree_counted_by_several_threads(api):
    """Counts that hand heavy chunks on, of one graph and tree, side by side on
    three streams: each has contexts of its own."""
    import threading

    import torch
    s, d, t = bursts(140_000, 5, 1)[:3]
    n = 14
    g, og = api.Graph(s, d, t, n), oracle.OracleGraph(s, d, t, n)
    tr = api.Tree(THREE[::4], 60)
    want = np.array([og.count(m, 60) for m in THREE[::4]], dtype=np.uint64)
    assert np.array_equal(api.count(g, tr), want)
    bad = []

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(12):
                if not np.array_equal(api.count(g, tr), want):
                    bad.append(k)

    th = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    [x.start() for x in th]
    [x.join() for x in th]
    assert not bad


@pytest.mark.parametrize("unit", [1, 2 ** 33])
@pytest.mark.parametrize("n_edges", [1, 255, 3000, 131_073])
def test_per_motif_searches_in_one_batch(api, n_edges, unit):
    """Per-motif mode over trees of every depth: one window and several, chunk
    lengths from 4 up, enough roots for chunks to be handed on; equal to the
    oracle, or for the largest graph to the searches launched one by one."""
    s, d, t = bursts(n_edges, 11, unit)
    g = api.Graph(s, d, t, 14)
    motifs = MIXED if n_edges < 10_000 else MIXED[:6] + THREE[::7]
    deltas = [9 * unit, 40 * unit]
    if n_edges < 10_000:
        og = oracle.OracleGraph(s, d, t, 14)
        want = np.array([[og.count(m, x) for m in motifs] for x in deltas], dtype=np.uint64)
    else:
        want = np.stack([api.count(g, api.Tree(motifs, x), mode="per_motif", chunk=128) for x in deltas])
    for i, x in enumerate(deltas):
        assert np.array_equal(api.count(g, api.Tree(motifs, x), mode="per_motif"), want[i])
    tr = api.Tree(motifs, deltas)
    assert np.array_equal(api.count(g, tr, mode="per_motif"), want)
    got, ms = api.count(g, tr, mode="per_motif", timed=True)[:2]
    assert np.array_equal(got, want) and ms > 0
