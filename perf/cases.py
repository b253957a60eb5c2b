"""Measured cases of the HP genotype-phenotype map library.

Each case is one call, or one short sequence of calls, as a program that maps
a lattice makes it: ground states of a window of sequences (blocked int8
form), the same with an energy table, reversal-canonical wide blocks, random
sampling and canonical sequences (dense int8 form), a captured batch of
several lattices, and the genotype-network passes over a complete map
(neighbour counts and components; the whole phi_pq matrix).

Structure handles and their device tables are built once per lattice and
kept, as every program of this library keeps them.  Inputs follow the seed:
the position of a window, the generator seed of a sampling run, or, for the
network passes, the real map of the lattice moved by a seeded point mutation
mask (an automorphism of the sequence cube) with its phenotype ids permuted.
Counters accumulate, so a pass zeroes them first, as a map step does.
"""
import random

import torch

import paper_2008_05612_amd as hp

HP1996 = (0, -10, -10, -23)          # the two-letter energies of Table 1, times 10
BOXES = {"4x4": (4, 4, 1), "5x5": (5, 5, 1), "6x6": (6, 6, 1), "2x3x4": (2, 3, 4),
         "3x3x3": (3, 3, 3)}

_handles = {}
_maps = {}


def _structs(box, table):
    """(handle, device workspace) of a lattice and "hp" or "hp1996" energies."""
    key = (box, table)
    if key not in _handles:
        s = hp.Structures(*BOXES[box], table=HP1996 if table == "hp1996" else None)
        _handles[key] = [s, None]
    h = _handles[key]
    if h[1] is None and torch.cuda.is_available():
        h[1] = h[0].workspace()
    return h


def listed():
    return [
        # a handful of sequences looked up: energies and gaps of 100 neighbours
        {"name": "lookup 3x3x3", "kind": "enumerate", "box": "3x3x3", "table": "hp", "n": 100,
         "align": 1, "emin": True, "threshold": 1},
        # the small square of the batch and test workloads, most of its map
        {"name": "window 4x4", "kind": "enumerate", "box": "4x4", "table": "hp", "n": 50001,
         "align": 1, "emin": False, "threshold": 0},
        # half of the 5x5 map in one launch, with energies
        {"name": "block 5x5", "kind": "enumerate", "box": "5x5", "table": "hp", "n": 1 << 24,
         "align": 1 << 17, "emin": True, "threshold": 0},
        # a ragged window of the cube with energies and an energy-gap threshold
        {"name": "window 3x3x3", "kind": "enumerate", "box": "3x3x3", "table": "hp",
         "n": 3000001, "align": 1, "emin": True, "threshold": 2},
        # one step of a streamed full 3x3x3 map (a quarter of it)
        {"name": "step 3x3x3", "kind": "enumerate", "box": "3x3x3", "table": "hp", "n": 1 << 25,
         "align": 1 << 17, "emin": False, "threshold": 0},
        # one step of the full 6x6 map from reversal-canonical wide blocks
        {"name": "step 6x6", "kind": "canonical", "box": "6x6", "n": 1 << 17, "keep": False},
        # a step of the cube's map with the energies of Table 1
        {"name": "step 3x3x3 table", "kind": "enumerate", "box": "3x3x3", "table": "hp1996",
         "n": 1 << 23, "align": 1 << 17, "emin": False, "threshold": 0},
        # one sampling launch of the paper's size
        {"name": "sample 3x3x3", "kind": "sample", "box": "3x3x3", "table": "hp", "n": 1 << 14},
        # the paper's timed workload at a production size: Table 1 energies on 6x6
        {"name": "sample 6x6 table", "kind": "sample", "box": "6x6", "table": "hp1996",
         "n": 1 << 20},
        # a captured batch over four lattices
        {"name": "batch", "kind": "batch", "n4": 50001, "n5": 1 << 20, "n24": 1 << 22,
         "n27": 1 << 19},
        # single-mutation statistics and neutral networks of the whole cube
        {"name": "network 3x3x3", "kind": "network", "box": "3x3x3"},
        # the whole phi_pq matrix of the cube: dense counts, then compressed rows
        {"name": "phi 3x3x3", "kind": "phi", "box": "3x3x3"},
    ]


def _log(rng, lo, hi):
    """A size between lo and hi, spread over its logarithm."""
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    kind = rng.choice(["enumerate", "enumerate", "enumerate", "enumerate", "table", "canonical",
                       "sample", "sample", "symmetric", "batch", "network", "phi"])
    if kind == "enumerate":
        box, top = rng.choice([("4x4", 60000), ("2x3x4", 1 << 23), ("5x5", 1 << 24),
                               ("3x3x3", 1 << 25), ("3x3x3", 1 << 25), ("6x6", 1 << 24)])
        n = _log(rng, 100, top)
        align = 1
        if n >= 1 << 18 and rng.random() < 0.5:      # as full-map drivers cut their ranges
            align = 1 << 17
            n = n >> 17 << 17
        return {"kind": "enumerate", "box": box, "table": "hp", "n": n, "align": align,
                "emin": rng.random() < 0.5, "threshold": rng.choice([0, 0, 0, 1, 2, 3])}
    if kind == "table":
        box, top = rng.choice([("4x4", 60000), ("2x3x4", 1 << 23), ("5x5", 1 << 23),
                               ("3x3x3", 1 << 23)])
        return {"kind": "enumerate", "box": box, "table": "hp1996", "n": _log(rng, 100, top),
                "align": 1, "emin": rng.random() < 0.5, "threshold": rng.choice([0, 0, 5, 10])}
    if kind == "canonical":
        box, top = rng.choice([("5x5", 10000), ("3x3x3", 1 << 15), ("6x6", 1 << 16)])
        return {"kind": "canonical", "box": box, "n": _log(rng, 1, top), "keep": box != "6x6"}
    if kind == "sample":
        box, table, top = rng.choice([("3x3x3", "hp", 1 << 20), ("3x3x3", "hp1996", 1 << 20),
                                      ("6x6", "hp", 1 << 20), ("6x6", "hp1996", 1 << 20),
                                      ("5x5", "hp1996", 1 << 21), ("4x4", "hp", 1 << 20)])
        return {"kind": "sample", "box": box, "table": table, "n": _log(rng, 16, top)}
    if kind == "symmetric":
        box, table, top = rng.choice([("6x6", "hp1996", 1 << 19), ("5x5", "hp", 1 << 21),
                                      ("3x3x3", "hp1996", 1 << 19)])
        return {"kind": "symmetric", "box": box, "table": table, "n": _log(rng, 1000, top),
                "keep": box != "6x6"}
    if kind == "batch":
        return {"kind": "batch", "n4": _log(rng, 100, 60000), "n5": _log(rng, 1000, 1 << 22),
                "n24": _log(rng, 1000, 1 << 22), "n27": _log(rng, 1000, 1 << 20)}
    box = rng.choice(["5x5", "2x3x4"])
    # several maps of one lattice differ by their seed only: `part` shifts it
    return {"kind": kind, "box": box, "part": rng.randrange(1 << 16)}


def _zeros(*shape):
    return torch.zeros(shape, dtype=torch.int64, device="cuda")


def _empty(n, dtype):
    return torch.empty(n, dtype=dtype, device="cuda")


def _window(rng, space, n, align):
    return rng.randrange((space - n) // align + 1) * align


def _outputs(s, n, emin, gap):
    return {"out": _empty(n, torch.int16), "emin": _empty(n, torch.int32) if emin else None,
            "gap": _empty(n, torch.uint8) if gap else None, "desig": _zeros(s.n_class),
            "nond": _zeros(1)}


def _moved_map(box, rng):
    """The lattice's real map under g -> g ^ mask with permuted phenotype ids."""
    s, ws = _structs(box, "hp")
    if box not in _maps:
        out = _empty(1 << s.N, torch.int16)
        hp.hp_enumerate(s, ws, hp.FORM_BLOCKED_I8, 0, 1 << s.N, out)
        _maps[box] = out
    gen = torch.Generator().manual_seed(rng.randrange(1 << 60))
    ids = torch.full((1 << 16,), -1, dtype=torch.int16)
    ids[:s.n_class] = torch.randperm(s.n_class, generator=gen).to(torch.int32).to(torch.int16)
    ids = ids.cuda()
    mask = rng.randrange(1 << s.N)
    out = torch.empty_like(_maps[box])
    step = 1 << 24
    for lo in range(0, 1 << s.N, step):
        hi = min(lo + step, 1 << s.N)
        g = torch.arange(lo, hi, device="cuda") ^ mask
        out[lo:hi] = ids[_maps[box][g].to(torch.int64) & 0xFFFF]
    return out


def prepare(case, seed):
    kind = case["kind"]
    rng = random.Random("%d %s" % (seed, kind))
    st = {"kind": kind, "case": case}
    if kind == "batch":
        jobs, outs = [], []
        for box, n, align in (("4x4", case["n4"], 1), ("5x5", case["n5"], 1),
                              ("2x3x4", case["n24"], 1), ("3x3x3", case["n27"], 1)):
            if n % (1 << 17) == 0:
                align = 1 << 17
            s, ws = _structs(box, "hp")
            lo = _window(rng, 1 << s.N, n, align)
            o = _outputs(s, n, False, False)
            jobs.append(hp.Job(s, ws, lo, lo + n, o["out"], None, o["desig"], o["nond"]))
            outs.append(o)
        bws = torch.zeros(hp._binding.batch_workspace_bytes(len(jobs)), dtype=torch.uint8,
                          device="cuda")
        st["outs"] = outs
        st["graph"] = hp.hp_graph_capture_batch(jobs, hp.FORM_BLOCKED_I8, bws)
        return st
    if kind in ("network", "phi"):
        box = case["box"]
        rng = random.Random("%d %s %d" % (seed, kind, case.get("part", 0)))
        s, _ = _structs(box, "hp")
        st["s"] = s
        st["map"] = _moved_map(box, rng)
        nq = s.n_class
        if kind == "phi":
            st["counts"] = _zeros(nq, nq + 1)
            st["row_ptr"] = _empty(nq + 1, torch.int64)
        else:
            st["phi_q"] = rng.randrange(nq)
            st["stats"] = [_zeros(nq), _zeros(nq), _zeros(nq), _zeros(nq + 1)]
            st["labels"] = _empty(1 << s.N, torch.int32)
            st["size"] = _empty(1 << s.N, torch.int32)
            st["ncomp"] = _empty(nq, torch.int32)
            st["largest"] = _empty(nq, torch.int32)
        return st
    table = case.get("table", "hp")
    s, ws = _structs(case["box"], table)
    st["s"], st["ws"], n = s, ws, case["n"]
    if kind == "enumerate":
        st["lo"] = _window(rng, 1 << s.N, n, case["align"])
        st["o"] = _outputs(s, n, case["emin"], case["threshold"] > 0)
    elif kind == "sample":
        st["seed"] = rng.randrange(1 << 62)
        st["o"] = _outputs(s, n, True, False)
        st["seqs"] = _empty(n, torch.int64)
    else:
        count = hp.hp_wide_block_count(s) if kind == "canonical" else hp.hp_canonical_count(s)
        st["lo"] = _window(rng, count, n, 1)
        st["o"] = {"out": None, "emin": None, "gap": None, "desig": _zeros(s.n_class),
                   "nond": _zeros(1)}
        if case["keep"]:        # the map of a whole lattice, filled at the scored places
            st["o"]["out"] = torch.full((1 << s.N,), -1, dtype=torch.int16, device="cuda")
    return st


def _zero(o):
    o["desig"].zero_()
    o["nond"].zero_()


def _results(o):
    return {k: v for k, v in o.items() if v is not None}


def run(state):
    kind, case = state["kind"], state["case"]
    if kind == "batch":
        for o in state["outs"]:
            _zero(o)
        state["graph"].launch()
        return [_results(o) for o in state["outs"]]
    s = state["s"]
    if kind == "network":
        for t in state["stats"]:
            t.zero_()
        neutral, deleterious, other, row = state["stats"]
        hp.hp_neighbors(s, state["map"], neutral, deleterious, other, state["phi_q"], row)
        hp.hp_components(s, state["map"], state["labels"], state["size"], state["ncomp"],
                         state["largest"])
        return state["stats"] + [state["labels"], state["size"], state["ncomp"], state["largest"]]
    if kind == "phi":
        state["counts"].zero_()
        hp.hp_phi_counts(s, state["map"], state["counts"])
        nnz = hp.hp_phi_sparse(s, state["counts"], state["row_ptr"])
        cols, vals = _empty(nnz, torch.int32), _empty(nnz, torch.int64)
        hp.hp_phi_sparse(s, state["counts"], state["row_ptr"], cols, vals)
        return [state["row_ptr"], cols, vals]
    ws, o, n = state["ws"], state["o"], case["n"]
    _zero(o)
    if kind == "enumerate":
        lo = state["lo"]
        if case["threshold"]:
            hp.hp_enumerate_gap(s, ws, hp.FORM_BLOCKED_I8, lo, lo + n, case["threshold"],
                                o["out"], o["emin"], o["gap"], o["desig"], o["nond"])
        else:
            hp.hp_enumerate(s, ws, hp.FORM_BLOCKED_I8, lo, lo + n, o["out"], o["emin"],
                            o["desig"], o["nond"])
    elif kind == "sample":
        hp.hp_sample(s, ws, hp.FORM_GEMM_I8, state["seed"], 0, n, 1, state["seqs"], o["out"],
                     o["emin"], None, o["desig"], o["nond"])
        return dict(_results(o), seqs=state["seqs"])
    elif kind == "canonical":
        hp.hp_enumerate_symmetric_wide(s, ws, state["lo"], state["lo"] + n, o["out"], None,
                                       o["desig"], o["nond"])
    else:
        hp.hp_enumerate_symmetric(s, ws, hp.FORM_GEMM_I8, state["lo"], state["lo"] + n, o["out"],
                                  None, o["desig"], o["nond"])
    return _results(o)


def exact(case, seed):
    """Every output is a whole number (phenotype ids, energies, counts), which
    stays equal; there is no rounding to compare in 64 bits."""
    return None


def _scored(s, n, per_seq_bytes):
    """Work of scoring n sequences: the contacts of every conformation read
    once (a bit per product row), the outputs written once; per pair nbp
    contact products and their sum."""
    return {"bytes": n * per_seq_bytes + s.n_conf * (s.K / 8 + 2) + 16 * s.n_class,
            "flops": 2.0 * s.nbp * n * s.n_conf}


def work(case):
    kind = case["kind"]
    if kind == "batch":
        w = [_scored(_structs(b, "hp")[0], case[k], 2)
             for b, k in (("4x4", "n4"), ("5x5", "n5"), ("2x3x4", "n24"), ("3x3x3", "n27"))]
        return {k: sum(x[k] for x in w) for k in ("bytes", "flops")}
    s = _structs(case["box"], case.get("table", "hp"))[0]
    total = 1 << s.N
    if kind == "network":
        # the map read once by each of the two calls; labels and sizes written
        return {"bytes": total * (2 + 2 + 4 + 4) + 8 * 6 * s.n_class, "flops": 2.0 * total * s.N}
    if kind == "phi":
        # the map, and the dense counts zeroed once and read once
        return {"bytes": total * 2 + 2 * 8 * s.n_class * (s.n_class + 1), "flops": total * s.N}
    if kind == "canonical":
        return _scored(s, case["n"] << 10, 4 if case["keep"] else 0)
    if kind == "symmetric":
        return _scored(s, case["n"], 4 if case["keep"] else 0)
    if kind == "sample":
        return _scored(s, case["n"], 2 + 4 + 8)
    return _scored(s, case["n"], 2 + 4 * case["emin"] + (1 if case["threshold"] else 0))
