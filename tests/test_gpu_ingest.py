"""The device-side graph ingest (time sort, lists, list ranks) at the sizes
where a pass can go wrong: around the sort's tile of 4,096 edges, vertex ids
around a digit of 8 bits, ties, self-loops, empty lists, 32- and 64-bit times.
Counts are whole numbers and must equal the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2507_14813_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api(oracle_mod):
    import torch
    assert torch.cuda.is_available(), "no GPU visible"
    from paper_2507_14813_amd import api
    api.lib()
    return api


MOTIFS = W.enumerate_motifs(3, 3) + [((0, 1),), ((0, 1), (1, 2), (3, 1), (3, 0))]


@pytest.mark.parametrize("n_edges,n_nodes", [
    (1, 2), (2, 2), (63, 255), (64, 256), (65, 257), (4095, 300), (4096, 65535), (4097, 65537),
    (70_001, 900), (300_000, 40_000)])
@pytest.mark.parametrize("wide", [False, True])
def test_unsorted_input_equals_oracle(api, n_edges, n_nodes, wide):
    print("ingest", n_edges, n_nodes, wide, flush=True)
    rng = np.random.default_rng(n_edges + wide)
    s = rng.integers(0, n_nodes, n_edges).astype(np.int32)
    d = np.where(rng.random(n_edges) < 0.3, rng.integers(0, min(8, n_nodes), n_edges),
                 rng.integers(0, n_nodes, n_edges)).astype(np.int32)       # a few hubs, some loops
    unit = 3 * 2 ** 31 if wide else 1
    t = (rng.integers(-40 * n_edges, 40 * n_edges + 1, n_edges) // 7).astype(np.int64) * unit - 9
    delta = 400 * unit
    og = oracle.OracleGraph(s, d, t, n_nodes)
    g = api.Graph(s, d, t, n_nodes)
    i = g.info()
    assert (i["self_loops"], i["t_min"], i["t_max"]) == (int((s == d).sum()), t.min(), t.max())
    want = np.array([og.count(m, delta) for m in MOTIFS], dtype=np.uint64)
    assert np.array_equal(api.count(g, api.Tree(MOTIFS, delta)), want)
    # edge ids come back in the caller's order
    m, e = api.enumerate_matches(g, api.Tree([((0, 1), (0, 1))], delta))
    a, b = e[:, 0], e[:, 1]
    assert len(a) == og.count(((0, 1), (0, 1)), delta)
    assert (s[a] == s[b]).all() and (d[a] == d[b]).all() and (s[a] != d[a]).all()
    assert (t[a] < t[b]).all() and (t[b] - t[a] <= delta).all()


@pytest.mark.parametrize("n_edges", [0, 1, 5000])
def test_only_self_loops_and_no_edges(api, n_edges):
    s = np.arange(n_edges, dtype=np.int32) % 7
    g = api.Graph(s, s, np.arange(n_edges, dtype=np.int64)[::-1].copy(), 7)
    assert g.info()["self_loops"] == n_edges
    assert not api.count(g, api.Tree(MOTIFS, 5)).any()
