"""The workloads this library is timed on, through its public Python API.

Each case is one call (or one batch, or one burst of requests) as a program
that uses the library makes it: single growths on every engine, the state
kinds and options used in earnest, the 4096-job batch and the request queue.
Outputs are the layer sizes of the growth (exact integers) and, where the
caller asks for them, the states of its layers.

``listed()`` names the cases, ``draw()`` gives more of the same ranges,
``prepare()`` makes a case's inputs (and the engine or queue its program
keeps), ``run()`` is one pass, ``work()`` the bytes and operations a pass
cannot do without, ``exact()`` the same outputs from a plain numpy search.
"""

from __future__ import annotations

import math

import numpy as np

from paper_2509_19162_amd import api
from paper_2509_19162_amd import inputs as I

#: States a caller reads back where a growth is too large to read whole.
EXPORT_CAP = 1 << 20

#: Room for layer sizes that every growth is given.
MAX_LAYERS = 512

#: Entry counts of the 4-bit coset start, by n (five colours at n = 14).
MULTISETS = {10: (2, 2, 2, 2, 2), 11: (3, 2, 2, 2, 2), 12: (3, 3, 2, 2, 2), 13: (3, 3, 3, 2, 2),
             14: (3, 3, 3, 3, 2), 15: (5, 5, 5), 16: (6, 5, 5)}


def listed():
    return [
        # One growth call on a small group, engine and buffers made and
        # dropped inside the call: a script trying one generating set.
        {"name": "call_s7", "kind": "call", "n": 7, "m": 2},
        # The same question asked again and again by a search over generating
        # sets that keeps its engine: one workgroup runs the whole job.
        {"name": "workgroup_s8", "kind": "workgroup", "n": 8, "m": 3},
        # S_8 with the adjacent transpositions from a random start, the
        # states of every layer read back (29 small layers, latency-bound).
        {"name": "layers_s8_coxeter", "kind": "layers", "n": 8, "family": "coxeter"},
        # An ordinary growth: S_10 under three random permutations and their
        # inverses, on an engine the program keeps.
        {"name": "engine_s10", "kind": "engine", "n": 10, "m": 3},
        # S_12 with the 11 prefix reversals, every layer kept on the device
        # (479,001,600 states), the first million states read back.
        {"name": "keep_s12_pancake", "kind": "keep", "n": 12, "family": "pancake"},
        # S_16 under L, R, X until a layer passes 2^29 states: a group too
        # large to finish, few generators, 64-bit ranks.
        {"name": "frontier_s16_lrx", "kind": "frontier", "n": 16, "frontier": 1 << 29},
        # The memory-saving engine on a group the serving queue sends to it.
        {"name": "bitmask_s13", "kind": "bitmask", "n": 13, "m": 2},
        # A set not closed under inverses: every earlier layer is subtracted.
        {"name": "directed_s11", "kind": "directed", "n": 11, "m": 2},
        # A Schreier coset graph of vectors with repeated entries (4 bits per
        # entry, packed keys): 14 positions, five colours, adjacent swaps.
        {"name": "coset_n14_coxeter", "kind": "coset", "n": 14, "family": "coxeter"},
        # A binary coset graph (1 bit per entry): 32 positions, 16 ones, LRX:
        # C(32,16) = 6.0e8 states in about 200 layers.
        {"name": "binary_n32_lrx", "kind": "binary", "n": 32, "ones": 16, "family": "lrx"},
        # The search over many generating sets: 4096 uneven jobs in a batch.
        {"name": "batch_4096", "kind": "batch", "jobs": 4096, "n_lo": 7, "n_hi": 10},
        # Serving: a burst of requests of mixed size and family, waited for.
        {"name": "queue_64", "kind": "queue", "requests": 64, "n_lo": 6, "n_hi": 11},
    ]


def draw(rng):
    while True:
        case = _draw(rng)
        if all({k: v for k, v in c.items() if k != "name"} != case for c in listed()):
            return case


def _draw(rng):
    kind = rng.choice(["call", "workgroup", "layers", "engine", "keep", "frontier", "bitmask", "directed", "coset",
                       "binary", "batch", "queue"])
    case = {"kind": kind}
    if kind == "layers":
        case.update(n=rng.randint(6, 9), family=rng.choice(["coxeter", "cyclic_coxeter", "star", "pancake", "lrx", "reversals"]))
    elif kind == "keep":
        case.update(n=rng.randint(10, 12), family=rng.choice(["pancake", "star", "coxeter", "cyclic_coxeter", "lrx"]))
    elif kind == "frontier":
        case.update(n=rng.randint(13, 16), frontier=int(2 ** rng.uniform(18, 28.9)))
    elif kind == "coset":
        case.update(n=rng.randint(10, 16), family=rng.choice(["coxeter", "lrx"]))
    elif kind == "binary":
        n = rng.randint(17, 32)
        case.update(n=n, ones=rng.randint(n // 3, n // 2), family="coxeter" if n <= 28 and rng.random() < 0.5 else "lrx")
    elif kind == "batch":
        lo = rng.randint(5, 8)
        case.update(jobs=int(2 ** rng.uniform(4, 12)), n_lo=lo, n_hi=rng.randint(lo, 10))
    elif kind == "queue":
        lo = rng.randint(5, 7)
        case.update(requests=rng.randint(4, 64), n_lo=lo, n_hi=rng.randint(lo + 1, 11))
    else:
        lo, hi = {"call": (5, 9), "workgroup": (6, 10), "engine": (9, 12), "bitmask": (10, 13), "directed": (8, 11)}[kind]
        n = rng.randint(lo, hi)
        case.update(n=n, m=2 if n == 13 else rng.randint(2, 4))
        if rng.random() < 0.5:  # a search cut short: no layer past this size is expanded
            case["frontier"] = int(math.factorial(n) ** rng.uniform(0.4, 0.9))
    return case


def _rng(case, seed):
    return np.random.Generator(np.random.PCG64([I.SEED, 7, int(seed), case["n"]]))


def _gens(case, seed):
    """The case's generator rows: a named family, or m random permutations
    (with their inverses unless the case is directed)."""
    if case["kind"] == "frontier":
        return I.lrx(case["n"])
    if "family" in case:
        return I.family(case["family"], case["n"])
    rows = I.random_perms_with_inverses(case["n"], case["m"], _rng(case, seed))
    return rows[: case["m"]] if case["kind"] == "directed" else rows


def _start(case, seed):
    """The case's start vector, or None for the identity."""
    n, r = case["n"], _rng(case, seed)
    if case["kind"] in ("layers", "keep", "frontier"):
        return [int(x) for x in r.permutation(n)]
    if case["kind"] == "coset":
        vec = [v for v, c in enumerate(MULTISETS[n]) for _ in range(c)]
        return [vec[i] for i in r.permutation(n)]
    if case["kind"] == "binary":
        vec = [0] * (n - case["ones"]) + [1] * case["ones"]
        return [vec[i] for i in r.permutation(n)]
    return None


def _options(case):
    kind, n = case["kind"], case["n"]
    opts = {"max_layers": MAX_LAYERS, "max_frontier": case.get("frontier")}
    if kind == "workgroup":
        opts["small_job"] = True
    elif kind == "layers":
        opts["export_layers"] = math.factorial(n)
    elif kind == "keep":
        opts.update(keep_all_layers=True, export_layers=min(EXPORT_CAP, math.factorial(n)))
    elif kind == "frontier":
        opts["export_layers"] = EXPORT_CAP
    elif kind == "bitmask":
        opts["bitmask"] = True
    elif kind == "directed":
        opts["allow_directed"] = True
    return opts


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        r = np.random.Generator(np.random.PCG64([I.SEED, 8, int(seed)]))
        jobs = []
        for _ in range(case["jobs"]):
            n = int(r.integers(case["n_lo"], case["n_hi"] + 1))
            jobs.append((n, I.random_perms_with_inverses(n, int(r.integers(2, 5)), r)))
        return {"kind": kind, "jobs": jobs}
    if kind == "queue":
        reqs = [I.serving_request(1000 * (int(seed) % 1000003) + i, n_lo=case["n_lo"], n_hi=case["n_hi"])
                for i in range(case["requests"])]
        return {"kind": kind, "requests": [(n, g) for n, _, g in reqs], "queue": api.GrowthQueue(max_active=256)}
    state = {"kind": kind, "n": case["n"], "gens": _gens(case, seed), "start": _start(case, seed),
             "options": _options(case)}
    if kind != "call":
        state["engine"] = api.Engine()
    return state


def _sizes(results):
    """Layer sizes of the growths, one row each, zeros after the last layer."""
    out = np.zeros((len(results), MAX_LAYERS), dtype=np.int64)
    for row, r in zip(out, results):
        row[: len(r.sizes)] = r.sizes
    return out


def run(state):
    kind = state["kind"]
    if kind == "call":
        sizes = api.growth(state["n"], state["gens"], **state["options"])
        return {"sizes": np.pad(np.array(sizes, dtype=np.int64), (0, MAX_LAYERS - len(sizes)))}
    if kind == "batch":
        return {"sizes": _sizes(api.growth_batch(state["jobs"], max_layers=MAX_LAYERS))}
    if kind == "queue":
        q = state["queue"]
        tickets = [q.submit(n, g, max_layers=MAX_LAYERS) for n, g in state["requests"]]
        return {"sizes": _sizes([q.wait(t) for t in tickets])}
    res = state["engine"].run(state["n"], state["gens"], start=state["start"], **state["options"])
    out = {"status": res.status, "sizes": _sizes([res])[0], "expanded": res.states_expanded,
           "candidates": res.candidates}
    if res.layers is not None:
        out["states"] = np.concatenate(res.layers)
    return out


def _states(case):
    """States a pass visits (each once), as far as the sizes tell: n!, the
    orbit of the start vector, or about four times the largest layer of a
    search cut short (LRX layers grow by a third)."""
    kind = case["kind"]
    if case.get("frontier"):
        return min(math.factorial(case["n"]), 4 * case["frontier"])
    if kind == "coset":
        return math.factorial(case["n"]) // math.prod(math.factorial(c) for c in MULTISETS[case["n"]])
    if kind == "binary":
        return math.comb(case["n"], case["ones"])
    return math.factorial(case["n"])


def work(case):
    """A growth has to write every state it reaches once and read it back
    once to expand it: 8 bytes each way, or one bit each way in the bitmap
    engines; every neighbour of an expanded state is formed once."""
    if case["kind"] in ("batch", "queue"):
        sizes = [math.factorial(n) for n in range(case["n_lo"], case["n_hi"] + 1)]
        states = sum(sizes) / len(sizes) * case["jobs" if case["kind"] == "batch" else "requests"]
        return {"bytes": states / 4 if case["kind"] == "batch" else 16 * states, "flops": 6 * states}
    states = _states(case)
    k = len(_gens(case, 0))
    per_state = 0.25 if case["kind"] in ("bitmask", "workgroup") else 16
    read_back = _options(case).get("export_layers", 0) * case["n"]
    return {"bytes": per_state * states + read_back, "flops": k * states}


def exact(case, seed):
    """The same outputs from a breadth-first search over numpy arrays, where
    that takes seconds."""
    if case["kind"] in ("batch", "queue", "frontier") or case.get("frontier") or _states(case) > 400_000:
        return None
    n, gens, opts = case["n"], [np.array(g) for g in _gens(case, seed)], _options(case)
    start = _start(case, seed)
    place = (16 if n <= 16 else 2) ** np.arange(n - 1, -1, -1, dtype=np.uint64)
    layer = np.array([list(range(n)) if start is None else start], dtype=np.uint8)
    seen = layer.astype(np.uint64) @ place
    layers, k = [layer], len({tuple(g) for g in gens if list(g) != list(range(n))})
    while True:
        cand = np.concatenate([layer[:, g] for g in gens])
        keys, first = np.unique(cand.astype(np.uint64) @ place, return_index=True)
        new = ~np.isin(keys, seen)
        if not new.any():
            break
        layer = cand[first[new]]
        seen = np.concatenate([seen, keys[new]])
        layers.append(layer)
    sizes = np.zeros(MAX_LAYERS, dtype=np.int64)
    sizes[: len(layers)] = [len(x) for x in layers]
    if case["kind"] == "call":
        return {"sizes": sizes}
    total = int(sizes.sum())
    out = {"status": 0, "sizes": sizes, "expanded": total, "candidates": total * k}
    if "export_layers" in opts:
        out["states"] = np.concatenate(layers)
    return out
