"""Levels large enough for the grid's own constructor kernels (blocks of more
than 16384 candidates), against the oracle: every count, the answer, and up to
200 stored rows of every level bit by bit.

Chunks of 50 001 and 20 011 candidates cut blocks inside rows, so first and
last rows of a piece are partial; operand levels of 2, 4, 5, ... rows beside
levels of thousands put either operand across the lanes.  All arithmetic is
bitwise: exact agreement.
"""
import pytest

import oracle

from paper_2305_18575_amd import instances
from test_gpu_parity import run_both

pytestmark = pytest.mark.gpu

# (generator, seed, p, le, alphabet, costs, max_cost, allowed errors, chunk)
SPECS = [
    ("type1", 1, 10, 5, "01", (1, 1, 1, 1, 1), 14, 0, 0),         # one word, keys in the slots
    ("type1", 2, 10, 4, "01", (1, 1, 1, 1, 1), 15, 0, 50001),     # few infixes: mostly duplicates
    ("type1", 7, 12, 7, "01", (1, 1, 10, 1, 1), 16, 0, 20011),    # two words
    ("type1", 8, 12, 8, "01", (1, 1, 1, 1, 1), 13, 2, 50001),     # four words, allowed errors
    ("type2", 5, 10, 6, "01", (1, 10, 1, 1, 1), 15, 0, 20011),
    ("type1", 4, 9, 5, "012", (1, 1, 1, 1, 1), 11, 0, 0),         # three characters
    ("type2", 3, 8, 5, "01", (2, 1, 3, 1, 1), 22, 0, 50001),
    ("type1", 6, 9, 5, "01", (1, 1, 1, 3, 1), 20, 0, 20011),      # mostly unions
    ("type1", 9, 9, 6, "01", (1, 2, 1, 4, 1), 23, 0, 50001),
]


@pytest.mark.parametrize("kind,seed,p,le,sigma,costs,max_cost,errors,chunk", SPECS)
def test_large_levels_equal_oracle(rei, kind, seed, p, le, sigma, costs, max_cost, errors, chunk):
    gen = instances.type1_instance if kind == "type1" else instances.type2_instance
    it = gen(seed, p, p, le, sigma=sigma, costs=costs, max_cost=max_cost)
    g, _ = run_both(rei, sigma, it.pos, it.neg, costs, max_cost, 4 << 30, max_errors=errors, chunk=chunk,
                    rows=True, row_limit=200)
    print(f"infixes={g.ic_size} words={g.cs_words} status={g.status} candidates={sum(g.candidates)}", flush=True)


@pytest.mark.parametrize("kind,seed,p,le,sigma,costs,max_cost,errors,chunk", [SPECS[0], SPECS[2], SPECS[7]])
def test_large_levels_after_hand_off(rei, kind, seed, p, le, sigma, costs, max_cost, errors, chunk):
    """The same levels continued on the grid after the one-workgroup solver
    stored the levels below (its rows' constructors are found from their
    back-pointers)."""
    it = instances.type1_instance(seed, p, p, le, sigma=sigma, costs=costs, max_cost=max_cost)
    h = rei.Instance(sigma, it.pos, it.neg, costs, max_cost, 4 << 30)
    h.set_batch_level(2000)
    g = rei.solve_batch([h])[0]
    o = oracle.Oracle(sigma, it.pos, it.neg, costs, max_cost, 1 << 40, 0, threads=8).solve()
    assert (g.status, g.cost, g.regex) == (o.status, o.cost, o.regex)
    for c in range(max_cost + 1):
        assert (g.unique_at(c), g.candidates_at(c)) == (o.unique[c], o.candidates[c]), c
    h.close()


@pytest.mark.parametrize("char_costs,max_cost", [([1, 2], 17), ([3, 1], 18)])
def test_large_levels_with_character_costs(rei, char_costs, max_cost):
    """Characters of different costs: a level may hold characters beside r?,
    r*, concatenations and unions."""
    costs = (1, 1, 1, 1, 1)
    it = instances.type1_instance(11, 9, 9, 5, costs=costs, max_cost=max_cost)
    h = rei.Instance("01", it.pos, it.neg, costs, max_cost, 4 << 30)
    h.set_char_costs(char_costs)
    g = h.solve()
    o = oracle.solve("01", it.pos, it.neg, costs=costs, max_cost=max_cost, char_costs=char_costs, threads=8)
    assert (g.status, g.cost, g.regex) == (o.status, o.cost, o.regex)
    for c in range(max_cost + 1):
        assert (g.unique_at(c), g.candidates_at(c)) == (o.unique[c], o.candidates[c]), c
    assert max(g.candidates) > 1 << 16
    h.close()
