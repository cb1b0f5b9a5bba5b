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
        self.peak = 0

    def alloc(self, n):
        import torch
        if self.bytes + n > self.limit or not self.calls:
            self.refused += 1
            return None
        self.calls -= 1
        p = torch.cuda.caching_allocator_alloc(n, 0)
        self.live[p] = n
        self.bytes += n
        self.peak = max(self.peak, self.bytes)
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


def type1(seed, p, le, costs, max_cost):
    return instances.type1_instance(seed, p, p, le, costs=costs, max_cost=max_cost)


def capped(it, max_cost):
    it.max_cost = min(it.max_cost, max_cost)
    return it


# (specification, cache bytes, device bytes): bytes that a search needs which
# allocates for one chunk after the other, chunks of a level doubling from 2^16
LIMITS = {
    "plain": (lambda: capped(instances.plain_instance(3), 12), 64 << 20, 82860),
    "single, 797 candidates": (lambda: instances.single_instance(8), 1 << 30, 263588),
    "single, 7092 candidates": (lambda: instances.single_instance(6), 1 << 30, 2078372),
    "single, 226958 candidates": (lambda: instances.single_instance(3, (1, 1, 5, 1, 2)), 1 << 30, 22029692),
    "one word, 41656 candidates": (lambda: type1(1, 10, 5, (1, 1, 1, 1, 1), 11), 4 << 30, 4020012),
    "one word, 1037685 candidates": (lambda: type1(13, 8, 6, (1, 1, 1, 1, 1), 14), 4 << 30, 66891192),
    "two words, 1473413 candidates": (lambda: type1(7, 12, 7, (1, 1, 10, 1, 1), 16), 4 << 30, 97469536),
    "16 words": (lambda: capped(instances.large_instance(0), 8), 1 << 30, 4677548),
    "32 words": (lambda: instances.wide_instance(3, 8), 1 << 30, 8876324),
}


@pytest.mark.parametrize("name", list(LIMITS))
def test_search_fits_the_memory_of_its_chunks(rei, name):
    """Nothing that is taken for speed alone (the one-workgroup start, large
    first chunks, buffers that grow ahead) turns a search away."""
    make, cache, limit = LIMITS[name]
    it = make()
    want = oracle_of([it], cache)
    with memory(rei) as m:
        m.limit = limit
        print(f"\n{name}: {limit} bytes", flush=True)
        h = handles(rei, [it], cache)[0]
        assert_equal([h.solve()], want, [it])
        print(f"{m.refused} allocations refused", flush=True)
        h.close()
        assert not m.live
        h = handles(rei, [it], cache)[0]
        m.limit = m.bytes
        with pytest.raises(rei.ReiError):  # with nothing at all it ends in an error
            h.solve()
        m.limit = 1 << 62
        assert_equal([h.solve()], want, [it])
        h.close()
        assert not m.live


@pytest.mark.parametrize("queue", [True, False])
def test_served_request_takes_nothing_ahead(rei, queue):
    """A server admits requests by the bytes they need.  One whose last level
    leaves its workgroup holds its arena (16 MB of 24-byte rows, a table of load
    at most 1/2) and the survivors of one chunk: 28 bytes a candidate."""
    it = instances.single_instance(3, (1, 1, 5, 1, 2))
    want = oracle_of([it], 1 << 30)
    rows = (16 << 20) // 24
    with memory(rei) as m:
        h = handles(rei, [it], 1 << 30)[0]
        srv = rei.Server(1 << 30, 64, 2, 2, queue=queue)
        res = srv.wait(srv.submit(h))[0]
        srv.close()
        need = 24 * rows + 8 * (1 << 21) + 28 * max(res.candidates) + (1 << 20)
        print(f"\npeak {m.peak}, need {need}", flush=True)
        assert_equal([res], want, [it])
        assert max(res.candidates) > 1 << 16 and 2 * (rows + 8192) <= 1 << 21 and sum(res.unique) < rows
        assert m.peak <= need
        h.close()


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


@pytest.mark.parametrize("calls", [0, 2, 7, 20, 60])
def test_batch_while_allocations_are_refused(rei, calls):
    """A batch whose searches leave their workgroups early, with so many
    allocations granted: it ends in an error or in the oracle's results, and
    the same instances give those once there is memory."""
    specs = instances.batched_instances(9, 12) + [capped(instances.large_instance(0), 8)]
    cache = 1 << 30
    want = oracle_of(specs, cache)
    with memory(rei) as m:
        hs = handles(rei, specs, cache)
        for h in hs:
            h.set_batch_level(300)
        m.calls = calls
        print(f"\n{calls} allocations", flush=True)
        try:
            got = rei.solve_batch(hs)
        except rei.ReiError as e:
            print(e, flush=True)
        else:
            assert_equal(got, want, specs)
        assert m.refused or m.calls > 0
        m.calls = 1 << 62
        for _ in range(2):
            assert_equal(rei.solve_batch(hs), want, specs)
        for h in hs:
            h.close()
        assert not m.live
