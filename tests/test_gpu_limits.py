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
