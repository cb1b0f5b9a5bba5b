"""The language cache fills inside a chunk of more than 2^18 candidates, whose
winners are ranked by the scan that is spread over the device: the first winner
that does not fit, the rows stored before it and the switch to OnTheFly mode,
against the oracle (exactly: all results are whole numbers and bytes).

A level of more than 2^18 candidates goes in chunks of 2^16, 2^19 and 2^22
candidates; the scan's blocks have 2^15 candidates each.  The caps put the first
winner that does not fit into the first, a middle and the last block of a chunk,
onto a chunk's first candidates, and onto the level's last ones.
"""
import pytest

import oracle

from paper_2305_18575_amd import instances

pytestmark = pytest.mark.gpu

FIRST, SECOND = 1 << 16, (1 << 16) + (1 << 19)  # where a level's second and third chunk begin
BLOCK = 1 << 15

# (seed, p, le, costs, max_cost): one word with the keys in the slots; two words
ONE = (13, 8, 6, (1, 1, 1, 1, 1), 14)
TWO = (7, 12, 7, (1, 1, 10, 1, 1), 16)
LEVEL = {ONE: (14, 1037685), TWO: (16, 1473413)}  # the level that fills the cache, its candidates

# rows that fit, and the range the first winner that does not fit lies in
FILLS = [
    (ONE, 178303, FIRST, FIRST + 8),
    (ONE, 188513, FIRST, FIRST + BLOCK),
    (ONE, 268544, FIRST + 8 * BLOCK, FIRST + 12 * BLOCK),
    (ONE, 301093, SECOND - BLOCK, SECOND),
    (ONE, 304194, SECOND, SECOND + 8),               # the second chunk's winners fit exactly: no room for the third's
    (ONE, 379385, 1037685 - BLOCK, 1037685),         # all but the last winner fit
    (TWO, 315174, FIRST, FIRST + 8),
    (TWO, 512970, FIRST + 8 * BLOCK, FIRST + 12 * BLOCK),
    (TWO, 567810, SECOND - BLOCK, SECOND),
    (TWO, 720070, 1473413 - BLOCK, 1473413),
]


def both(rei, spec, cap, max_errors=0, on_the_fly=False):
    seed, p, le, costs, max_cost = spec
    it = instances.type1_instance(seed, p, p, le, costs=costs, max_cost=max_cost)
    words = 1 if instances.n_infixes(it.pos + it.neg) <= 64 else 2
    print(f"\ncase: {spec} rows {cap} errors {max_errors} on the fly {on_the_fly}", flush=True)
    h = rei.Instance("01", it.pos, it.neg, costs, max_cost, cap * (8 * words + 8))
    if max_errors:
        h.set_max_errors(max_errors)
    if on_the_fly:
        h.set_on_the_fly(True)
    g = h.solve()
    o = oracle.solve("01", it.pos, it.neg, costs=costs, max_cost=max_cost, row_cap=cap, max_errors=max_errors,
                     threads=8, on_the_fly=on_the_fly)
    assert (g.status, g.cost, g.regex) == (o.status, o.cost, o.regex)
    for c in range(max_cost + 1):
        assert (g.unique_at(c), g.candidates_at(c)) == (o.unique[c], o.candidates[c]), c
    h.close()
    return o


@pytest.mark.parametrize("spec,cap,lo,hi", FILLS)
def test_cache_fills_in_a_large_chunk(rei, spec, cap, lo, hi):
    o = both(rei, spec, cap)
    level, total = LEVEL[spec]
    assert o.status == "OUT_OF_MEMORY" and lo <= o.candidates[level] - 1 < hi <= total


@pytest.mark.parametrize("spec,cap,lo,hi", FILLS)
def test_on_the_fly_from_a_large_chunk(rei, spec, cap, lo, hi):
    o = both(rei, spec, cap, on_the_fly=True)
    level, total = LEVEL[spec]
    assert o.candidates[level] == total and sum(o.unique) == cap  # full before the level's end


# an answer at candidate 671 229 of its level, in its third chunk, after 563 295 stored rows
ANSWER = (14, 9, 6, (1, 1, 1, 1, 1), 15)


@pytest.mark.parametrize("cap,status", [(1 << 24, "OK"), (563295, "OK"), (563294, "OUT_OF_MEMORY"),
                                        (545000, "OUT_OF_MEMORY"), (400000, "OUT_OF_MEMORY")])
@pytest.mark.parametrize("on_the_fly", [False, True])
def test_answer_around_the_fill_point(rei, cap, status, on_the_fly):
    o = both(rei, ANSWER, cap, max_errors=2, on_the_fly=on_the_fly)
    assert o.status == ("OK" if on_the_fly else status)
    if o.status == "OK":
        assert (o.cost, o.candidates[15]) == (15, 671230)
