"""rei_tune_grid times each parameter set as later solves run it."""
import pytest

from paper_2305_18575_amd import instances

pytestmark = pytest.mark.gpu

# 60 solves: best of three for the values in force and 6 + 3 + 5 + 5 others
SOLVES = 60


@pytest.mark.parametrize("own_first", [0, 1 << 10])
def test_tuner_chunks_levels_as_the_table_does(rei, own_first, tmp_path):
    """Every level here has at most four of the smallest first chunks tried
    (2^14), so an instance that takes its first chunk from the table has one
    chunk per level whichever is in force, and so must each timed solve; a first
    chunk the caller set on the instance holds again afterwards."""
    it = instances.type1_instance(1, 10, 10, 5, costs=(1, 1, 1, 1, 1), max_cost=11)
    h = rei.Instance("01", it.pos, it.neg, it.costs, 11, 1 << 30)
    k = rei.KERNEL_CLASSES.index("insert_survivors")

    def insertions(call):
        h.set_profiling(False)
        h.set_profiling_class("insert_survivors")
        out = call()
        return h.kernel_stats(k)[0], out

    one, r = insertions(h.solve)
    assert 1 << 15 < max(r.candidates) <= 4 << 14
    h.set_grid_tuning(own_first, 0, 0, 0)
    own, _ = insertions(h.solve)
    assert (own > one) == (own_first != 0)
    try:
        tuned, chosen = insertions(lambda: rei.tune_grid([h]))
        print(f"\n{one} insertions a solve, {tuned} in the tuner's {SOLVES}: {chosen}", flush=True)
        assert tuned == SOLVES * one
        assert insertions(h.solve)[0] == own
    finally:
        back = tmp_path / "defaults.json"
        back.write_text('{"grid": [{"words": 1, "first_chunk": 65536, "chunk_max": 16777216, "concat_wg": 2048, '
                        '"concat_xi": 16}]}\n')
        rei.tune_load(str(back))
    h.close()
