"""Device memory that the calls take and keep, seen from a registered allocator
that counts it and can be given a limit."""
import numpy as np
import pytest

import oracle
from paper_2507_14813_amd import workloads as W

pytestmark = pytest.mark.gpu

THREE = W.enumerate_motifs(3, 3)
MB = 1 << 20


@pytest.fixture(scope="module")
def api(oracle_mod):
    import torch
    assert torch.cuda.is_available(), "no GPU visible"
    from paper_2507_14813_amd import api
    api.lib()
    return api


_kept = []   # callbacks stay callable as long as anything they allocated may live


class Accounting:
    """torch's allocator with the bytes handed out counted (live, peak) and, with
    `limit`, refused beyond it."""

    def __init__(self, api):
        import torch
        self.api, self.limit, self.live, self.peak, self.sizes = api, None, 0, 0, {}

        def alloc(nbytes, stream, ctx):
            if self.limit is not None and self.live + nbytes > self.limit:
                return None
            p = int(torch.cuda.caching_allocator_alloc(int(nbytes), torch.cuda.current_device(),
                                                       int(stream or 0)))
            self.sizes[p] = int(nbytes)
            self.live += int(nbytes)
            self.peak = max(self.peak, self.live)
            return p

        def release(ptr, stream, ctx):
            self.live -= self.sizes.pop(int(ptr))
            torch.cuda.caching_allocator_delete(int(ptr))

        self.callbacks = (api._ALLOC_FN(alloc), api._RELEASE_FN(release))
        _kept.append(self)

    def __enter__(self):
        self.api.use_torch_allocator()
        self.saved = self.api._callbacks
        self.set(self.callbacks)
        return self

    def __exit__(self, *exc):
        self.set(self.saved)

    def set(self, callbacks):
        assert self.api.lib().mg_set_allocator(callbacks[0], callbacks[1], None) == 0
        self.api._callbacks = callbacks

    def used_by(self, call):
        """Peak bytes that a call takes beyond what was live before it."""
        before = self.peak = self.live
        out = call()
        return out, self.peak - before


def run_of_one_pair(n_edges):
    z = np.zeros(n_edges, np.int32)
    return z, z + 1, np.arange(n_edges, dtype=np.int64)


def test_counts_keep_no_context_buffer(api):
    """A count that hands chunks on takes its 16 MB for the call only, and other
    counts never: trees hold their tables alone."""
    n = 140_000
    with Accounting(api) as mem:
        g = api.Graph(*run_of_one_pair(n), 2)
        base = mem.live
        same = [((0, 1),) * 3]
        trees = [api.Tree(same, w) for w in (20, 30, 40, 50, 60)]
        for tr, w in zip(trees, (20, 30, 40, 50, 60)):
            print("contexts", w, flush=True)
            want = sum(min(w, i) * (min(w, i) - 1) // 2 for i in range(n))
            got, used = mem.used_by(lambda: api.count(g, tr))
            assert got.tolist() == [want] and 16 * MB <= used < 17 * MB
            got, used = mem.used_by(lambda: api.count(g, tr, mode="per_motif"))
            assert got.tolist() == [want] and used < 17 * MB
            assert mem.live - base < MB
        two = api.Tree([((0, 1), (1, 0)), ((0, 1), (0, 1))], 30)
        cost = np.zeros(n, np.uint64)
        for call in (lambda: api.count(g, two), lambda: api.count(g, trees[0], stats=True),
                     lambda: api.count(g, trees[0], max_chunks=10 ** 6),
                     lambda: api.count(g, two, mode="per_motif")):
            assert mem.used_by(call)[1] < MB
        assert mem.used_by(lambda: api.count(g, trees[0], root_cost=True))[1] < MB + cost.nbytes
        # without memory for contexts the waves keep their chunks
        mem.limit = mem.live + 8 * MB
        want = sum(min(60, i) * (min(60, i) - 1) // 2 for i in range(n))
        assert api.count(g, trees[-1]).tolist() == [want]
        assert api.count(g, trees[-1], mode="per_motif").tolist() == [want]
        b = api.Batch([g, g], [trees[-1], two], item_roots=64)
        assert b.count()[0].tolist() == [want]
        mem.limit = None
        del b, g, trees, two, tr, call
        import gc
        gc.collect()
        assert mem.live == 0
