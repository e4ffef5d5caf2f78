"""Calls at the limits of what the entry points take: launch settings far above
the defaults.  Whole numbers, equal to the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2507_14813_amd import workloads as W

pytestmark = pytest.mark.gpu

THREE = W.enumerate_motifs(3, 3)


@pytest.fixture(scope="module")
def api(oracle_mod):
    import torch
    assert torch.cuda.is_available(), "no GPU visible"
    from paper_2507_14813_amd import api
    api.lib()
    return api


def uniform(n_edges, n_nodes, span, seed):
    rng = np.random.default_rng(seed)
    return (rng.integers(0, n_nodes, n_edges).astype(np.int32),
            rng.integers(0, n_nodes, n_edges).astype(np.int32),
            np.sort(rng.integers(0, span, n_edges)).astype(np.int64))


@pytest.mark.parametrize("blocks,chunk", [(16_384, 65_536), (20_000, 65_536), (70_000, 16_384)])
def test_failing_claims_do_not_wrap_a_queue_head(api, blocks, chunk):
    """Every wave's last claim fails and still moves the head by a chunk: here
    they move it past 2^32, and no root may be searched twice for it."""
    s, d, t = uniform(5000, 60, 40_000, 3)
    g, og = api.Graph(s, d, t, 60), oracle.OracleGraph(s, d, t, 60)
    motifs = THREE[::7] + [((0, 1),)]
    tr = api.Tree(motifs, 300)
    want = np.array([og.count(m, 300) for m in motifs], dtype=np.uint64)
    print("heads", blocks, chunk, flush=True)
    assert np.array_equal(api.count(g, tr), want)
    assert np.array_equal(api.count(g, tr, blocks=blocks, chunk=chunk, queues=1), want)
    assert np.array_equal(api.count_noalloc(g, tr, blocks=blocks, chunk=chunk, queues=1), want)
    cur = api.Cursor()
    assert np.array_equal(api.count(g, tr, blocks=blocks, chunk=chunk, queues=1, cursor=cur), want)
    assert cur.done and list(cur.head) == [5000] + [0] * 7


def run_of_one_pair(n_edges, unit=1):
    z = np.zeros(n_edges, np.int32)
    return z, z + 1, np.arange(n_edges, dtype=np.int64) * unit


def repetitions(n_edges, k, w):
    """Matches of the k-edge repetition of a pair that has one edge per time
    unit, within w units: the first edge and k - 1 of the (at most w) after it."""
    after = np.minimum(w, np.arange(n_edges)[::-1]).astype(object)
    out = 1
    for i in range(k - 1):
        out = out * (after - i) // (i + 1)
    return int(np.sum(np.where(after >= k - 1, out, 0)))


# 300,000 roots with `w` later edges each: at three edges more than (64 w - 512) /
# 256 contexts for each of the 4,688 chunks, at four (64 w - 256) / 64, 2^18 and
# more in all
FULL = {3: 300, 4: 64}


@pytest.mark.parametrize("unit", [1, 2 ** 33])
@pytest.mark.parametrize("k", [3, 4])
def test_counts_that_fill_the_context_buffer(api, k, unit):
    n, w = 300_000, FULL[k]
    g = api.Graph(*run_of_one_pair(n, unit), 2)
    same = lambda j: ((0, 1),) * j
    want = repetitions(n, k, w)
    print("full buffer", k, unit, flush=True)
    assert api.count(g, api.Tree([same(k)], w * unit)).tolist() == [want]
    assert api.count(g, api.Tree([same(k)], [w * unit, 3 * unit])).tolist() == \
        [[want], [repetitions(n, k, 3)]]
    motifs = [same(2), same(k), ((0, 1), (1, 0), (0, 1))]
    assert api.count(g, api.Tree(motifs, w * unit), mode="per_motif").tolist() == \
        [repetitions(n, 2, w), want, 0]


@pytest.mark.parametrize("first", ["shallow", "empty", "one edge"])
@pytest.mark.parametrize("k", [3, 4])
def test_a_batch_that_fills_the_context_buffer(api, k, first):
    """The first job of the batch hands nothing on: a two-edge tree, or a graph
    without (or with one) edges."""
    n, w = 300_000, FULL[k]
    g, same = api.Graph(*run_of_one_pair(n), 2), lambda j: ((0, 1),) * j
    if first == "shallow":
        g0, t0, want0 = g, api.Tree([same(2)], 5), repetitions(n, 2, 5)
    else:
        g0, t0, want0 = api.Graph(*run_of_one_pair(int(first == "one edge")), 2), api.Tree([same(k)], w), 0
    print("full buffer, batch", k, first, flush=True)
    want = [[want0], [repetitions(n, k, w)]]
    graphs, trees = [g0, g], [t0, api.Tree([same(k)], w)]
    assert [x.tolist() for x in api.count_batch(graphs, trees)] == want
    b = api.Batch(graphs, trees, item_roots=64)
    for _ in range(3):
        assert [x.tolist() for x in b.count()] == want


@pytest.mark.parametrize("n_motifs,k", [(450, 5), (510, 4), (512, 5)])
def test_batches_of_thousands_of_counters(api, n_motifs, k):
    """Trees of up to MG_MAX_QUERIES counters in a batch: the counters of a
    workgroup's waves and their level buffers share 160 KB."""
    motifs = list(dict.fromkeys(tuple(m) for m in W.random_extension_motifs(4 * n_motifs, (k,), 6, 9)))
    motifs = motifs[:n_motifs]
    deltas = [10 * (i + 1) for i in range(8)]
    tr = api.Tree(motifs, deltas)
    assert tr.info()["n_distinct"] == n_motifs and tr.info()["depth"] == k
    s, d, t = uniform(800, 12, 4000, 5)
    g, og = api.Graph(s, d, t, 12), oracle.OracleGraph(s, d, t, 12)
    print("counters", n_motifs * 8, k, flush=True)
    want = api.count(g, tr)
    for i in (0, 3, 7):
        assert want[i][::37].tolist() == [og.count(m, deltas[i]) for m in motifs[::37]]
    small = api.Tree(THREE, 30)
    want0 = np.array([og.count(m, 30) for m in THREE], dtype=np.uint64)
    for got in (api.count_batch([g, g], [small, tr]), api.Batch([g, g], [small, tr], item_roots=64).count()):
        assert np.array_equal(got[0], want0) and np.array_equal(got[1], want)


def test_epochs_of_two_edge_trees_hand_contexts_on(api):
    """Whole-list windows of a two-edge tree, most waves without a chunk: the
    busy ones hand on what is left, as in deeper trees."""
    s, d, t = uniform(40_000, 3000, 40_000, 7)
    g, og = api.Graph(s, d, t, 3000), oracle.OracleGraph(s, d, t, 3000)
    motifs = [((0, 1), (2, 3)), ((0, 1), (1, 2))]
    for unit in (1, 2 ** 33):
        g = api.Graph(s, d, t * unit, 3000)
        want = np.array([[og.count(m, x) for m in motifs] for x in (100, 2000)], dtype=np.uint64)
        for delta, exp in ((2000 * unit, want[1]), ([100 * unit, 2000 * unit], want)):
            for epochs in (2, 16):
                log = np.zeros(epochs, np.int64)
                print("two-edge epochs", unit, delta, epochs, flush=True)
                got = api.count(g, api.Tree(motifs, delta), epoch_idle=1, max_epochs=epochs, epoch_contexts=log)
                assert np.array_equal(got, exp) and log[0] > 0 and log[-1] == 0


def test_enumeration_into_too_little_room_ends_its_search(api):
    """A capacity far below the matches: nothing is written, the total is that
    of the count, and it does not take the time of enumerating everything (here
    over 3,000 times the count's work: 2 * 10^8 matches)."""
    import ctypes
    import time
    n, w, k = 300_000, 50, 3
    g, tree = api.Graph(*run_of_one_pair(n), 2), api.Tree([((0, 1),) * k], w)
    total = repetitions(n, k, w)
    L, m = api.lib(), ctypes.c_int64(0)

    def call(capacity):
        rec = np.full((max(capacity, 1), 6), -7, np.int32)
        t0 = time.perf_counter()
        assert L.mg_enumerate(g.handle, tree.handle, None, rec.ctypes.data, capacity, ctypes.byref(m)) == 0
        dt = time.perf_counter() - t0
        assert m.value == total and (rec == -7).all()
        return dt

    print("little room", total, flush=True)
    for capacity in (1, 63, 64, 5000, 1_000_000):
        call(capacity)
    assert min(call(5000) for _ in range(5)) < 0.02


def test_enumeration_with_room_for_every_match(api):
    """Capacities at the total and around it, each record once; a tree whose
    only motif is one edge (matches of the roots themselves)."""
    import ctypes
    L = api.lib()
    for k, w, n in ((1, 0, 1000), (2, 3, 5000), (4, 6, 2000)):
        g, tree, m = api.Graph(*run_of_one_pair(n), 2), api.Tree([((0, 1),) * k], w), ctypes.c_int64(0)
        total = repetitions(n, k, w)
        for capacity in (total - 1, total, total + 1, 4 * total):
            rec = np.full((capacity, 6), -7, np.int32)
            assert L.mg_enumerate(g.handle, tree.handle, None, rec.ctypes.data, capacity,
                                  ctypes.byref(m)) == 0
            assert m.value == total
            if capacity < total:
                assert (rec == -7).all()
            else:
                got = rec[:total]
                assert (rec[total:] == -7).all() and (got[:, 0] == 0).all() and (got[:, 1 + k:] == -1).all()
                assert len(set(map(tuple, got[:, 1:1 + k].tolist()))) == total
                assert (np.diff(got[:, 1:1 + k], axis=1) > 0).all() and (got[:, k] - got[:, 1] <= w).all()


def test_autotuner_starts_from_the_defaults(api, tmp_path):
    """What mg_tune names as the defaults is what a count without settings runs
    (chunk 0: the launch chooses), also from a cache that says 64."""
    s, d, t = uniform(30_000, 200, 20_000, 4)
    g, tr, cache = api.Graph(s, d, t, 200), api.Tree(THREE[::5], 300), tmp_path / "tune.jsonl"
    print("tune", flush=True)
    r = api.tune(g, tr, cache=str(cache))
    assert r["chunk"] in (0, 128, 256) and r["from_cache"] == 0
    line = cache.read_text()
    assert '"chunk": %d,' % r["chunk"] in line
    cache.write_text(line.replace('"chunk": %d,' % r["chunk"], '"chunk": 64,'))
    r2 = api.tune(g, tr, cache=str(cache))
    assert r2["from_cache"] == 1 and r2["chunk"] == 0
    kw = {k: r2[k] for k in ("blocks", "chunk", "queues", "leaf_scan")}
    assert np.array_equal(api.count(g, tr, **kw), api.count(g, tr))


@pytest.mark.parametrize("unit", [1, 2 ** 33])
def test_handed_on_chunks_equal_the_oracle(api, unit):
    """Enough roots and long enough windows for chunks to be handed on (64 roots
    with about 25 entries in each of their lists, 768 candidates and more): one
    window and two, per motif and in a batch, three- and four-edge trees."""
    n, nodes = 140_000, 250
    s, d, t = uniform(n, nodes, 10 * n, 6)
    og = oracle.OracleGraph(s, d, t, nodes)
    w = 25 * int(t[-1]) * nodes // n
    three = THREE[::6]
    four = [((0, 1), (1, 2), (2, 0), (0, 1)), ((0, 1), (0, 2), (2, 1), (1, 0))]
    g = api.Graph(s, d, t * unit, nodes)
    for motifs in (three, three[:2] + four):
        want = np.array([[og.count(m, x) for m in motifs] for x in (w // 3, w)], dtype=np.uint64)
        trees = [api.Tree(motifs, x * unit) for x in (w // 3, w)]
        multi = api.Tree(motifs, [w // 3 * unit, w * unit])
        print("handed on", unit, len(motifs), flush=True)
        assert np.array_equal(np.stack([api.count(g, x) for x in trees]), want)
        assert np.array_equal(api.count(g, multi), want)
        assert np.array_equal(np.stack([api.count(g, x, mode="per_motif") for x in trees]), want)
        assert np.array_equal(api.count(g, multi, mode="per_motif"), want)
        assert np.array_equal(np.stack(api.count_batch([g, g], trees)), want)
        assert np.array_equal(api.count_batch([g, g], [trees[0], multi])[1], want)
        b = api.Batch([g, g], [multi, trees[1]])
        for _ in range(3):
            x, y = b.count()
            assert np.array_equal(x, want) and np.array_equal(y, want[1])
