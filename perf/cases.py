"""The calls a user of the library makes, as timed cases.

Each case is one pass through the public entry points of
``paper_1804_09741_amd.motifs`` on seeded synthetic digraphs (the recipes of
``paper_1804_09741_amd.inputs``).  A case's ``op`` names the call:

  count        one blocking count of one loaded graph, histogram on the host
  run          one pass of a prepared batch into a device histogram; the
               batch is one graph and ``randoms`` degree-preserving random
               versions of it (0: the graph alone)
  static       one allocation-free count into a device histogram
  count7       H_7 of a graph and its random versions (classes by code)
  ensemble     the significance pipeline: make the random versions, count
               them all in one batch, z-score every class on the device
  serve        a burst of requests through the continuous-batching server
  cold         a program's start: open a context, build the class table,
               count one graph, close
"""

import math

import numpy as np
import torch

from paper_1804_09741_amd import inputs as I
from paper_1804_09741_amd import motifs as M

SWITCHES_PER_ARC = 10
K7_ROWS = 1 << 16  # the most classes of one graph that count7 returns by default


def listed():
    return [
        # The smallest count: a triad census of a small uniform graph (n = 200,
        # m = 800).  All latency: allocations, launches, copies.
        {"name": "k3_count_er", "op": "count", "k": 3, "recipe": "er", "n": 200, "m": 800},
        # One mid-size hub-heavy graph at k = 4, counted again and again
        # through a prepared batch (a parameter study on one graph).
        {"name": "k4_run", "op": "run", "k": 4, "recipe": "chung_lu", "n": 2000, "m": 10000,
         "gamma": 2.2, "cap": 200, "recip": 0.2, "randoms": 0},
        # The call for programs that may not allocate, on one graph of the
        # k = 5 study's size; always by enumeration.
        {"name": "k5_static", "op": "static", "k": 5, "recipe": "chung_lu", "n": 1000, "m": 3000,
         "gamma": 2.1, "cap": 200, "recip": 0.1},
        # A significance study's counting pass at k = 5: the original and 100
        # random versions in one launch.
        {"name": "k5_batch101", "op": "run", "k": 5, "recipe": "chung_lu", "n": 1000, "m": 3000,
         "gamma": 2.1, "cap": 200, "recip": 0.1, "randoms": 100},
        # The same study end to end: random versions made on the device,
        # batch prepared, counted, every class z-scored.
        {"name": "k5_ensemble", "op": "ensemble", "k": 5, "recipe": "chung_lu", "n": 1000,
         "m": 3000, "gamma": 2.1, "cap": 200, "recip": 0.1, "randoms": 100},
        # k = 6, one sparse power-law graph: few units for the whole chip.
        {"name": "k6_run", "op": "run", "k": 6, "recipe": "powerlaw", "n": 700, "m": 1500,
         "randoms": 0},
        # k = 6, that graph and 30 random versions: the benchmark's step.
        {"name": "k6_batch31", "op": "run", "k": 6, "recipe": "powerlaw", "n": 700, "m": 1500,
         "randoms": 30},
        # k = 6 at the dense end of the request stream (m = 6 n, degrees to 60):
        # the largest single graphs that fit the on-chip marks.
        {"name": "k6_run_dense", "op": "run", "k": 6, "recipe": "chung_lu", "n": 5000,
         "m": 30000, "gamma": 2.3, "cap": 60, "recip": 0.0, "randoms": 0},
        # k = 6 past the on-chip marks limit, an odd vertex count: sorted
        # lists and marks in device memory.
        {"name": "k6_run_lists", "op": "run", "k": 6, "recipe": "sparse", "n": 131073, "m": 0,
         "randoms": 0},
        # k = 7 on a sparse graph and 15 random versions.
        {"name": "k7_batch16", "op": "count7", "k": 7, "recipe": "powerlaw", "n": 700, "m": 1500,
         "randoms": 15},
        # 32 requests of mixed k and size at once through the server.
        {"name": "serve_burst32", "op": "serve", "k": 0, "recipe": "stream", "n": 1500, "m": 0,
         "requests": 32},
        # A command-line count at k = 6: the 2^30-entry class table is built,
        # used once and dropped.
        {"name": "k6_cold", "op": "cold", "k": 6, "recipe": "powerlaw", "n": 700, "m": 1500},
    ]


def _between(rng, lo, hi):
    """A whole number spread over [lo, hi] by its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["count", "run", "run", "run", "batch", "batch", "static", "count7",
                     "ensemble", "serve", "lists", "cold"])
    if op == "serve":
        return {"op": "serve", "k": 0, "recipe": "stream", "n": _between(rng, 200, 1500), "m": 0,
                "requests": rng.randint(3, 32)}
    if op == "lists":
        return {"op": "run", "k": rng.choice([4, 5, 6]), "recipe": "sparse",
                "n": _between(rng, 8193, 131073), "m": 0, "randoms": 0}
    if op == "cold":
        n = _between(rng, 100, 700)
        return {"op": "cold", "k": rng.choice([4, 5, 6]), "recipe": "powerlaw", "n": n,
                "m": int(n * rng.uniform(1.6, 2.2))}
    if op == "count7" or (op == "batch" and rng.random() < 0.5):
        # sparse power-law graphs and their random versions (k = 6, 7)
        n = _between(rng, 100, 700)
        c = {"op": "run" if op == "batch" else op, "k": 6 if op == "batch" else 7,
             "recipe": "powerlaw", "n": n, "m": int(n * rng.uniform(1.6, 2.2)),
             "randoms": rng.randint(1, 30 if op == "batch" else 15)}
        return c
    if op in ("batch", "ensemble"):
        n = _between(rng, 100, 1000)
        return {"op": "run" if op == "batch" else op, "k": rng.choice([3, 4, 5]),
                "recipe": "chung_lu", "n": n, "m": int(n * rng.uniform(1.5, 3.0)),
                "gamma": round(rng.uniform(2.0, 2.6), 3), "cap": 200,
                "recip": round(rng.uniform(0.0, 0.3), 3), "randoms": _between(rng, 3, 100)}
    # one graph: the request stream's ranges
    k = rng.choice([3, 4, 5]) if op == "static" else rng.choice([3, 4, 5, 6])
    n = _between(rng, 100, 1000 if op == "static" else 5000)
    c = {"op": op, "k": k, "recipe": "chung_lu", "n": n,
         "m": int(n * rng.uniform(2.0, 3.0 if op == "static" else 6.0)),
         "gamma": round(rng.uniform(2.0 if k <= 5 else 2.3, 2.6), 3),
         "cap": 200 if k <= 5 else 60,
         "recip": round(rng.choice([0.0, rng.uniform(0.0, 0.3)]), 3)}
    if op == "run":
        c["randoms"] = 0
    return c


def _graph(case, seed):
    """The case's digraph as an out-adjacency CSR pair."""
    rng = np.random.default_rng([int(seed) & 0xFFFFFFFF, case["n"], case["m"]])
    if case["recipe"] == "er":
        return I.er_digraph(case["n"], case["m"], rng)
    if case["recipe"] == "powerlaw":
        return I.powerlaw_out_digraph(case["n"], case["m"], 2.5, 60, rng)
    if case["recipe"] == "sparse":
        return I.sparse_powerlaw_digraph(case["n"], 2.5, 60, rng)
    return I.chung_lu_digraph(case["n"], case["m"], case["gamma"], case["cap"], case["recip"], rng)


def _request(case, seed, i):
    """The graph of request i: the benchmark stream's ranges (n uniform up to
    the case's, m = 2 n .. 6 n, degrees to 200, or 60 at k = 6); the sizes k
    take turns."""
    rng = np.random.default_rng([int(seed) & 0xFFFFFFFF, case["n"], i])
    n = int(rng.integers(100, case["n"] + 1))
    return I.chung_lu_digraph(n, int(n * rng.uniform(2.0, 6.0)), rng.uniform(2.0, 2.6),
                              60 if 3 + i % 4 == 6 else 200, 0.0, rng)


_context = None


def _ctx():
    """The program's one device context, with its class tables."""
    global _context
    if _context is None:
        _context = M.Context(0)
    return _context


class _State:
    """What the caller's program holds between passes; handles are freed
    with it."""

    def __init__(self, case, seed):
        self.case = case
        self.seed = int(seed)
        self.graphs, self.batch, self.server = [], None, None
        self.table = self.d_hist = self.d_z = None
        self.requests = []

    def __del__(self):
        if self.server is not None:
            self.server.stop()
        if self.batch is not None:
            self.batch.free()
        for g in self.graphs:
            g.free()


def prepare(case, seed):
    s = _State(case, seed)
    op = case["op"]
    if op == "cold":
        s.csr = _graph(case, seed)
        return s
    ctx = _ctx()
    if op == "serve":
        for i in range(case["requests"]):
            s.graphs.append(ctx.load_graph(*_request(case, seed, i)))
            s.requests.append((s.graphs[-1], 3 + i % 4))
        for k in range(3, 7):
            ctx.table(k)
        s.server = ctx.server()
        return s
    s.graphs.append(ctx.load_graph(*_graph(case, seed)))
    if case.get("randoms", 0) and op != "ensemble":
        made, _ = ctx.randomise(s.graphs[0], case["randoms"], s.seed, SWITCHES_PER_ARC)
        s.graphs.extend(made)
    if op == "count7":
        # the classes of all graphs as one table (graph, place, code and count)
        s.classes = np.zeros((len(s.graphs), K7_ROWS, 2), dtype=np.uint64)
        return s
    s.table = ctx.table(case["k"])
    if op in ("run", "static", "ensemble"):
        rows = 1 + case.get("randoms", 0)
        s.d_hist = torch.zeros((rows, s.table.num_classes), dtype=torch.int64, device="cuda:0")
        torch.cuda.synchronize()
    if op == "ensemble":
        s.d_z = torch.zeros((3, s.table.num_classes), dtype=torch.float64, device="cuda:0")
        torch.cuda.synchronize()
    if op == "run":
        s.batch = ctx.batch(s.graphs, s.table)
    return s


def run(s):
    op = s.case["op"]
    if op == "run":
        s.batch.run(s.d_hist, torch.cuda.current_stream())
        return s.d_hist
    if op == "count":
        hist, total = _ctx().count(s.graphs[0], s.table)
        return {"hist": hist, "total": total}
    if op == "static":
        _ctx().count_static(s.graphs[0], s.table, s.d_hist, torch.cuda.current_stream())
        return s.d_hist
    if op == "count7":
        out, totals, _ = _ctx().count7(s.graphs)
        for row, (codes, counts) in zip(s.classes, out):
            row[:len(codes), 0], row[:len(codes), 1] = codes, counts
        return {"classes": s.classes, "totals": totals}
    if op == "ensemble":
        ctx, stream = _ctx(), torch.cuda.current_stream()
        made, accepted = ctx.randomise(s.graphs[0], s.case["randoms"], s.seed, SWITCHES_PER_ARC)
        batch = ctx.batch([s.graphs[0]] + made, s.table)
        batch.run(s.d_hist, stream)
        ctx.significance(s.d_hist, s.table.num_classes, s.d_z, stream)
        batch.free()
        for g in made:
            g.free()
        return {"accepted": accepted, "hist": s.d_hist, "z": s.d_z}
    if op == "serve":
        tickets = [s.server.submit(g, k) for g, k in s.requests]
        return [s.server.wait(t, k)[0] for t, (_, k) in zip(tickets, s.requests)]
    ctx = M.Context(0)  # cold
    graph = ctx.load_graph(*s.csr)
    table = ctx.table(s.case["k"])
    hist, total = ctx.count(graph, table)
    out = {"hist": hist, "total": total, "codes": table.class_codes(),
           "cores": table.core_mult()}
    graph.free()
    ctx.close()
    return out


def work(case):
    """Inputs read once and outputs written once.  Counting is integer work;
    it has no floating operations."""
    k = case["k"]
    arcs = case["m"] or int(1.77 * case["n"])
    csr = 4 * (case["n"] + 1) + 4 * arcs
    if case["op"] == "serve":
        n, r = case["n"] / 2, case["requests"]
        hist = 8 * sum(M.NUM_CLASSES.values()) / 4
        return {"bytes": int(r * (4 * n + 16 * n + hist)), "flops": 0}
    graphs = 1 + case.get("randoms", 0)
    if case["op"] == "count7":
        return {"bytes": graphs * (csr + 16 * 10 * case["n"]), "flops": 0}
    size = graphs * (csr + 8 * M.NUM_CLASSES[k])
    if case["op"] == "ensemble":
        size += 2 * graphs * csr + 8 * 3 * M.NUM_CLASSES[k] + 8 * graphs * M.NUM_CLASSES[k]
    if case["op"] == "cold":
        size += 4 * 2 ** (k * (k - 1)) + 5 * M.NUM_CLASSES[k]
    return {"bytes": size, "flops": 0}


def exact(case, seed):
    """Counts are whole numbers.  Only the z-scores are computed numbers, and
    a plain 64-bit count of a hundred random graphs takes minutes."""
    return None
