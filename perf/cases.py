"""The work that programs have this framework do, as timed cases.

Each case names a family of specifications (seeded synthetic ones, as the tests
and the benchmark draw them), how many of them one pass solves, the search's
options, and the public entry point that the pass goes through.  The seed picks
the specifications, so another seed is other inputs of the same family.

A search's results are whole numbers and bytes: per specification the status,
the minimal cost, the printed expression, and the languages and candidates of
every cost level.  Every one of them is exact, so ``exact`` gives no value.
"""
import json

import numpy as np

import paper_2305_18575_amd as rei
from paper_2305_18575_amd import instances as I

MB = 1 << 20
STATUS_CODES = {name: code for code, name in rei.STATUS.items()}


def _case(family, entry, count=1, costs="1,1,1,1,1", max_cost=12, cache_mb=1024, le=0, p=10,
          max_errors=0, on_the_fly=False):
    return {"family": family, "entry": entry, "count": count, "costs": costs, "max_cost": max_cost,
            "cache_mb": cache_mb, "le": le, "p": p, "max_errors": max_errors, "on_the_fly": on_the_fly}


def listed():
    return [
        # one small question asked once: staged, solved, printed, given back
        dict(_case("plain", "one_shot", max_cost=12, cache_mb=64), name="plain one-shot"),
        # one mid-sized staged specification (2-4 words per language), an easy or a deep one
        dict(_case("single", "solve", count=8, max_cost=18), name="single solves"),
        # the benchmark's flagship: a few large ternary specifications at once (8-16 words)
        dict(_case("large", "batch", count=4, max_cost=12, cache_mb=8192), name="large batch"),
        # a mid-sized batch under the two cost functions of the single configuration
        dict(_case("single", "batch", count=64, max_cost=18), name="single batch"),
        # many small uneven specifications in one call
        dict(_case("batched", "batch", count=512, max_cost=12, cache_mb=256), name="batched call"),
        # the same kind of set captured once and replayed
        dict(_case("batched", "graph", count=512, max_cost=12, cache_mb=256), name="batched replay"),
        # a serving burst: plain, large and single requests in a mix
        dict(_case("mix", "server", count=48, max_cost=10), name="served burst"),
        # the widest languages (32 words), a bounded search
        dict(_case("wide", "solve", max_cost=10, cache_mb=8192), name="wide solve"),
        # a deep search over one-word languages, as the paper's Table 1 has them
        dict(_case("type1", "solve", le=6, max_cost=21, cache_mb=25600), name="deep 1-word solve"),
        # a deep search over two-word languages under an uneven cost function
        dict(_case("type1", "solve", le=7, p=12, costs="1,1,10,1,1", max_cost=21, cache_mb=25600),
             name="deep 2-word solve"),
        # four-word languages, an expression that may misclassify two examples
        dict(_case("type1", "solve", le=8, p=12, max_cost=17, max_errors=2, cache_mb=25600),
             name="allowed-error solve"),
        # a cache too small for the search, which goes on without storing
        dict(_case("type1", "solve", le=6, max_cost=20, cache_mb=64, on_the_fly=True), name="on-the-fly solve"),
    ]


def draw(rng):
    """One more case: a family, and sizes and options over that family's range."""
    kind = rng.choice(["plain", "single", "large", "batched", "mix", "wide", "type1", "type1", "type2", "type2"])
    if kind == "plain":
        entry = rng.choice(["one_shot", "solve", "batch"])
        count = 1 if entry == "one_shot" else int(round(2 ** rng.uniform(0, 6)))
        return _case("plain", entry, count=count, cache_mb=rng.choice([16, 64, 256]), max_cost=rng.randint(8, 14))
    if kind == "single":
        entry = rng.choice(["solve", "batch", "one_shot"])
        count = int(round(2 ** (rng.uniform(2, 6) if entry == "batch" else rng.uniform(0, 3))))
        return _case("single", entry, count=count, max_cost=rng.randint(8, 18), cache_mb=rng.choice([64, 1024]))
    if kind == "large":
        return _case("large", rng.choice(["solve", "batch"]), count=rng.randint(1, 4), max_cost=rng.randint(7, 12),
                     cache_mb=rng.choice([1024, 8192]))
    if kind == "batched":
        return _case("batched", rng.choice(["batch", "graph"]), count=int(round(2 ** rng.uniform(3, 9))),
                     max_cost=rng.randint(8, 12), cache_mb=rng.choice([64, 256]))
    if kind == "mix":
        return _case("mix", "server", count=rng.randint(4, 48), max_cost=rng.randint(7, 10))
    if kind == "wide":
        return _case("wide", rng.choice(["solve", "batch"]), max_cost=rng.randint(6, 10), cache_mb=8192)
    le = rng.randint(4, 8)
    costs, top = rng.choice([("1,1,1,1,1", 23 - le // 2), ("1,1,10,1,1", 21), ("1,10,1,1,1", 20), ("1,1,5,1,2", 22),
                             ("10,10,10,1,10", 100), ("20,20,20,5,30", 260)])
    max_cost = rng.randint(int(0.75 * top), top - le // 4)
    if kind == "type1" and rng.random() < 0.4:
        return _case("type1", "solve", le=le, p=rng.randint(8, 12), costs=costs, max_cost=max_cost,
                     cache_mb=rng.choice([4, 16, 64]), on_the_fly=rng.random() < 0.6)
    return _case(kind, rng.choice(["solve", "one_shot"]), le=le, p=rng.randint(8, 12), costs=costs,
                 max_cost=max_cost, cache_mb=25600, max_errors=rng.choice([0, 0, 1, 3]))


def _specs(case, seed):
    """The specifications of one state and each one's cache size in bytes."""
    rng = np.random.Generator(np.random.PCG64(seed))
    family, cap = case["family"], case["max_cost"]
    costs = tuple(int(x) for x in case["costs"].split(","))
    out = []
    while len(out) < case["count"]:
        k = len(out)
        sub = int(rng.integers(0, 1 << 30))
        cache = case["cache_mb"] * MB
        kind = family
        if family == "mix":  # the serving mix: 60 % plain, 30 % large, 10 % single
            kind = ("plain", "large", "plain", "plain", "single", "plain", "large", "plain", "large", "plain")[k % 10]
            cache = 64 * MB if kind == "plain" else 1024 * MB
        if kind == "plain":
            it = I.plain_instance(sub)
        elif kind == "single":
            it = I.single_instance(sub, (1, 1, 1, 1, 1) if k % 2 == 0 else (1, 1, 5, 1, 2))
        elif kind == "large":
            it = I.large_instance(sub)
        elif kind == "wide":
            try:
                it = I.wide_instance(sub, cap)
            except ValueError:  # this seed's specification is not that wide
                continue
        elif kind == "batched":
            it = I.batched_instances(sub, 1)[0]
        else:
            gen = I.type1_instance if kind == "type1" else I.type2_instance
            it = gen(sub, case["p"], case["p"], case["le"], costs=costs, max_cost=cap)
        out.append((it, min(it.max_cost, cap), cache))
    return out


def prepare(case, seed):
    """What a program holds before the call: strings for a one-shot call, else
    staged specifications, and the captured graph or the server it keeps."""
    specs = _specs(case, seed)
    state = {"case": case, "specs": specs}
    if case["entry"] == "one_shot":
        return state
    insts = []
    for it, max_cost, cache in specs:
        h = rei.Instance(it.alphabet, it.pos, it.neg, it.costs, max_cost, cache)
        if case["max_errors"]:
            h.set_max_errors(case["max_errors"])
        if case["on_the_fly"]:
            h.set_on_the_fly(True)
        insts.append(h)
    state["insts"] = insts
    if case["entry"] == "graph":
        state["graph"] = rei.BatchGraph(insts)
    elif case["entry"] == "server":
        state["server"] = rei.Server(hbm_budget=60 << 30)
    return state


def _outputs(results, max_cost):
    """Everything a search returns, as arrays over the specifications.  No
    search goes beyond level max_cost, and no expression of that cost takes
    more than four bytes per unit of it."""
    levels, chars = max_cost + 1, 4 * max_cost
    n = len(results)
    head = np.array([(STATUS_CODES[r.status], r.cost, r.first_level, r.total_unique, r.ic_size, r.cs_words)
                     for r in results], dtype=np.int64)
    text = [r.regex.encode() for r in results]
    return {"head": head, "regex": _padded(b"".join(text), [len(t) for t in text], n, chars, np.uint8),
            "unique": _padded([u for r in results for u in r.unique], [len(r.unique) for r in results], n,
                              levels, np.int64),
            "candidates": _padded([u for r in results for u in r.candidates],
                                  [len(r.candidates) for r in results], n, levels, np.int64)}


def _padded(values, lengths, n, width, dtype):
    """n rows of `width` values, row k holding the next lengths[k] of `values`."""
    flat = np.frombuffer(values, dtype=dtype) if isinstance(values, bytes) else np.array(values, dtype=dtype)
    lengths = np.array(lengths, dtype=np.int64)
    if lengths.max() > width:
        raise ValueError(f"a result has more than {width} values")
    out = np.zeros((n, width), dtype=dtype)
    out[np.arange(width) < lengths[:, None]] = flat
    return out


def _solve_all(state):
    case, entry = state["case"], state["case"]["entry"]
    if entry == "one_shot":
        return [rei.solve(it.alphabet, it.pos, it.neg, it.costs, max_cost, cache, max_errors=case["max_errors"],
                          on_the_fly=case["on_the_fly"]) for it, max_cost, cache in state["specs"]]
    if entry == "solve":
        return [h.solve() for h in state["insts"]]
    if entry == "batch":
        return rei.solve_batch(state["insts"])
    if entry == "graph":
        return state["graph"].run()
    tickets = [state["server"].submit(h) for h in state["insts"]]
    return [state["server"].wait(t)[0] for t in tickets]


def run(state):
    return _outputs(_solve_all(state), state["case"]["max_cost"])


_work_memo = {}


def work(case):
    """The bytes of one pass, from one solved example of the case (a search's
    size shows only by running it): every language found is written once to
    the cache with its back-pointer and its slot, and read once as an operand.
    The arithmetic is bitwise: no floating-point operation is needed."""
    key = json.dumps({k: v for k, v in case.items() if k != "name"}, sort_keys=True)
    if key not in _work_memo:
        state = prepare(dict(case, entry="solve"), 1)
        results = _solve_all(state)
        _work_memo[key] = float(sum(sum(r.unique) * (16 * r.cs_words + 16) + 8 * r.cs_words for r in results))
        for h in state["insts"]:
            h.close()
    return {"bytes": max(_work_memo[key], 1.0), "flops": 0.0}


def exact(case, seed):
    """No floating-point output: all results are whole numbers and bytes."""
    return None
