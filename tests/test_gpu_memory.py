"""Device memory that runs out: what a call does when an allocation fails, and
that the next call, with memory there again, gives the oracle's results.

The memory comes from torch's caching allocator through rei_set_allocator, whose
callbacks refuse on request."""
import contextlib

import pytest

from oracle_runs import mismatch, solve_many
from paper_2305_18575_amd import instances

pytestmark = pytest.mark.gpu


class Memory:
    """Live bytes of the callbacks' blocks; more than `limit` bytes, and
    allocations beyond the next `calls`, are refused."""

    def __init__(self):
        self.live, self.bytes, self.limit, self.calls, self.refused = {}, 0, 1 << 62, 1 << 62, 0

    def alloc(self, n):
        import torch
        if self.bytes + n > self.limit or not self.calls:
            self.refused += 1
            return None
        self.calls -= 1
        p = torch.cuda.caching_allocator_alloc(n, 0)
        self.live[p] = n
        self.bytes += n
        return p

    def free(self, p):
        import torch
        self.bytes -= self.live.pop(p)
        torch.cuda.caching_allocator_delete(p)


@contextlib.contextmanager
def memory(rei):
    m = Memory()
    rei.set_allocator(m.alloc, m.free)
    try:
        yield m
    finally:
        rei.set_allocator(None, None)


def handles(rei, specs, cache):
    return [rei.Instance(i.alphabet, i.pos, i.neg, i.costs, i.max_cost, cache) for i in specs]


def oracle_of(specs, cache):
    return solve_many([(i.alphabet, i.pos, i.neg, i.costs, i.max_cost, cache) for i in specs], workers=8, threads=1)


def assert_equal(got, want, specs):
    for k, (g, o) in enumerate(zip(got, want)):
        assert mismatch(g, o, specs[k].max_cost) is None, (k, mismatch(g, o, specs[k].max_cost))


@pytest.mark.parametrize("calls", [0, 1, 3, 8])
def test_graph_replay_after_a_failed_one(rei, calls):
    """Instances that outgrow a replay's arenas are solved outside it, in
    buffers that are then replaced.  When that fails midway, no replay starts
    until every descriptor names buffers that exist."""
    specs = instances.batched_instances(5, 60)
    cache = 1 << 30
    want = oracle_of(specs, cache)
    with memory(rei) as m:
        hs = handles(rei, specs, cache)
        g = rei.BatchGraph(hs, 1 << 16)
        print(f"\n{m.bytes} bytes after the capture, {calls} more allocations", flush=True)
        m.calls = calls
        for _ in range(2):
            with pytest.raises(rei.ReiError):
                g.run()
        assert m.refused
        m.calls = 1 << 62
        for rep in range(3):
            print(f"replay {rep}", flush=True)
            assert_equal(g.run(), want, specs)
        g.close()
        for h in hs:
            h.close()
        assert not m.live
