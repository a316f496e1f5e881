"""The calls a user of the library makes, as cases that can be timed and compared.

A case is one call (for serving: one burst of requests) through the Python binding, with
inputs that stay on the device as a user's program keeps them.  Sizes follow the seeded
workloads of paper_2212_00574_amd/inputs.py; draw() spreads over the same ranges.
"""
import math

import numpy as np
import torch

from paper_2212_00574_amd import binding as kzb

RESULT = ("status", "rounds", "equals_input", "passes", "surviving_vertices", "surviving_edges", "input_edges",
          "edge_tests")
DOM_RESULT = ("status", "sweeps", "deleted_vertices", "deleted_edges", "input_edges", "events")


def listed():
    return [
        # the smallest call: a hundred vertices as a byte matrix, latency and launches only
        {"name": "dense 100", "kind": "dense", "n": 100, "k": 4, "p": 0.5},
        # the ordinary single graph, bit rows, nothing removed
        {"name": "rows 3000", "kind": "rows", "n": 3000, "k": 10, "p": 0.6, "plant": True, "call": "blocking"},
        # the largest single graph, bit rows (the headline workload)
        {"name": "rows 20000", "kind": "rows", "n": 20000, "k": 20, "p": 0.3, "plant": False, "call": "blocking"},
        # a served-size sparse graph whose removals cascade over many rounds, ragged classes
        {"name": "rows cascade 5003", "kind": "rows", "n": 5003, "k": 23, "p": 0.14, "plant": False,
         "call": "blocking"},
        # a large sparse graph as CSR, uneven classes
        {"name": "csr 100000", "kind": "csr", "n": 100000, "k": 30, "m": 2500000},
        # many small graphs in one launch
        {"name": "batch 4096", "kind": "batch", "graphs": 4096, "less": 0},
        # a smaller batch with cliques two below the number of colour classes
        {"name": "batch colours 512", "kind": "batch", "graphs": 512, "less": 2},
        # a burst of served requests of all sizes, both lanes
        {"name": "serve 96", "kind": "serve", "requests": 96, "top": 12000},
        # both dominance reductions on one graph of the evaluation's recipe
        {"name": "dominance 1100", "kind": "dominance", "n": 1100, "mode": "both"},
        # the clique search on a graph that holds one planted clique
        {"name": "clique 12x90", "kind": "clique", "k": 12, "size": 90, "p": 0.4},
        # the struction around vertex 0
        {"name": "struction 1000", "kind": "struction", "n": 1000, "p": 0.1},
        # the upstream colouring of an uncoloured graph
        {"name": "colouring 3000", "kind": "colouring", "n": 3000, "p": 0.3},
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["dense", "rows", "rows", "rows", "csr", "batch", "batch", "serve", "dominance", "clique",
                       "struction", "colouring"])
    if kind == "dense":
        return {"kind": kind, "n": log_int(30, 1500), "k": rng.randint(2, 8), "p": round(rng.uniform(0.4, 0.8), 3)}
    if kind == "rows":
        n = log_int(200, 20000)
        k = rng.randint(5, 30)
        # the large sparse end (long cascades) stops where a call would take most of a second
        p = rng.uniform(0.1 if n <= 3000 else 0.2, 0.9)
        return {"kind": kind, "n": n, "k": k, "p": round(p, 3), "plant": rng.random() < 0.3,
                "call": rng.choice(["blocking", "blocking", "async"])}
    if kind == "csr":
        n = log_int(2000, 100000)
        return {"kind": kind, "n": n, "k": rng.choice([4, rng.randint(5, 40), 70]), "m": n * rng.randint(6, 25)}
    if kind == "batch":
        return {"kind": kind, "graphs": log_int(16, 2048), "less": rng.choice([0, 0, 1, 2])}
    if kind == "serve":
        return {"kind": kind, "requests": rng.randint(8, 96), "top": log_int(1000, 12000)}
    if kind == "dominance":
        return {"kind": kind, "n": log_int(100, 1100), "mode": rng.choice(["vertex", "edge", "both"])}
    if kind == "clique":
        return {"kind": kind, "k": rng.randint(4, 12), "size": rng.randint(8, 90),
                "p": round(rng.uniform(0.2, 0.4), 3)}
    if kind == "struction":
        return {"kind": kind, "n": log_int(100, 1000), "p": round(rng.uniform(0.03, 0.1), 3)}
    n = log_int(300, 20000)
    return {"kind": kind, "n": n, "p": round(min(0.6, rng.uniform(0.2, 1.0) * 900.0 / n), 4)}


# ------------------------------------------------------------------ inputs
_HANDLE, _SERVER = [], []


def _kz():
    if not _HANDLE:
        _HANDLE.append(kzb.Kernelizer(0))
    return _HANDLE[0]


def _server():
    """The one server a serving program keeps, on a stream of its own."""
    if not _SERVER:
        _SERVER.append(kzb.Server(_kz(), 4 << 30, max_slots=512, stream=torch.cuda.Stream()))
        _SERVER[0].configure(split_n=1024)
    return _SERVER[0]


def _near_equal(n, k):
    base, extra = divmod(n, k)
    return [base + (1 if c < extra else 0) for c in range(k)]


def _words(sizes):
    return sum((s + 63) // 64 for s in sizes)


def _gen(sizes, p, seed, gid, plant, rows, colour):
    """Class-major bit rows and colours of one seeded graph, written at two device addresses."""
    planted = None
    if plant:
        start = np.concatenate([[0], np.cumsum(sizes)[:-1]])
        rng = np.random.default_rng([seed, gid, 7])
        planted = [int(a + rng.integers(0, s)) for a, s in zip(start, sizes)]
    kzb.kz_gen_bitset(_kz().ctx, sizes, p, seed, gid, planted, rows, _words(sizes), colour,
                      torch.cuda.current_stream().cuda_stream)


def _rows_graph(sizes, p, seed, gid=0, plant=False):
    n = sum(sizes)
    rows = torch.empty((n, _words(sizes)), dtype=torch.int64, device="cuda")
    colour = torch.empty(n, dtype=torch.int32, device="cuda")
    _gen(sizes, p, seed, gid, plant, rows.data_ptr(), colour.data_ptr())
    return rows, colour


def _symmetric(n, p, gen):
    a = torch.rand((n, n), generator=gen, device="cuda") < p
    a = torch.triu(a, 1)
    return a | a.T


def _plain_rows(adj):
    """Bit rows int64 [n, ceil(n/64)] of a boolean matrix."""
    n = adj.shape[0]
    words = (n + 63) // 64
    full = torch.zeros((n, words * 64), dtype=torch.bool, device="cuda")
    full[:, :n] = adj
    b = full.view(n, words * 8, 8).to(torch.uint8)
    b = (b << torch.arange(8, dtype=torch.uint8, device="cuda")).sum(2, dtype=torch.uint8)
    return b.contiguous().view(torch.int64)


def _dominance_graph(n, gen):
    """The evaluation's recipe: a path through all vertices, n(n-5)/2 edges, some vertices favoured."""
    t = torch.rand(n, generator=gen, device="cuda", dtype=torch.float64) ** 2
    i, j = torch.triu_indices(n, n, 1, device="cuda")
    off = j != i + 1
    i, j = i[off], j[off]
    weight = (1 - t[i]) * (1 - t[j]) + 1e-3
    key = torch.rand(i.numel(), generator=gen, device="cuda", dtype=torch.float64).log() / weight
    absent = n * (n - 1) // 2 - n * (n - 5) // 2
    drop = torch.topk(key, absent).indices
    adj = ~torch.eye(n, dtype=torch.bool, device="cuda")
    adj[i[drop], j[drop]] = False
    adj[j[drop], i[drop]] = False
    return adj


def _pairs_of_cliques(n, k, colour, count, gen):
    """Keys lo * n + hi of the pairs inside `count` cliques of one random vertex per class."""
    by_class = torch.sort(colour, stable=True).indices
    sizes = torch.bincount(colour, minlength=k)
    start = torch.cumsum(sizes, 0) - sizes
    pick = (torch.rand((count, k), generator=gen, device="cuda") * sizes).to(torch.int64)
    v = by_class[start + torch.minimum(pick, sizes - 1)]
    i, j = torch.triu_indices(k, k, 1, device="cuda")
    a, b = v[:, i].reshape(-1), v[:, j].reshape(-1)
    return torch.unique(torch.minimum(a, b) * n + torch.maximum(a, b))


def _sparse(n, k, m, gen):
    """m distinct edges: a clique of the wanted size per 2000 vertices, the rest uniform pairs between classes."""
    colour = torch.randint(0, k, (n,), generator=gen, device="cuda", dtype=torch.int32)
    colour[:k] = torch.arange(k, dtype=torch.int32, device="cuda")
    planted = _pairs_of_cliques(n, k, colour, n // 2000, gen)
    count = int(m * 1.3 * k / (k - 1)) + 256
    a = torch.randint(0, n, (count,), generator=gen, device="cuda")
    b = torch.randint(0, n, (count,), generator=gen, device="cuda")
    ok = colour[a] != colour[b]
    a, b = a[ok], b[ok]
    key = torch.unique(torch.minimum(a, b) * n + torch.maximum(a, b))
    key = key[~torch.isin(key, planted)]
    key = key[torch.randperm(key.numel(), generator=gen, device="cuda")[:m - planted.numel()]]
    key = torch.cat([planted, key])
    lo, hi = key // n, key % n
    both = torch.sort(torch.cat([lo * n + hi, hi * n + lo])).values
    src, dst = both // n, both % n
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    row_ptr[1:] = torch.cumsum(torch.bincount(src, minlength=n), 0)
    return row_ptr, dst.to(torch.int32), colour


def _struction_graph(n, p, gen):
    """A random graph whose vertex 0 has a set degree and whose other part B a set edge count (the result's
    size depends on both)."""
    adj = _symmetric(n, p, gen)
    perm = torch.randperm(n - 1, generator=gen, device="cuda") + 1
    degree = int(round(p * (n - 1)))
    adj[0, :] = False
    adj[0, perm[:degree]] = True
    b = perm[degree:]
    i, j = torch.triu_indices(b.numel(), b.numel(), 1, device="cuda")
    keep = torch.topk(torch.rand(i.numel(), generator=gen, device="cuda"), int(round(p * i.numel()))).indices
    inside = torch.zeros((b.numel(), b.numel()), dtype=torch.bool, device="cuda")
    inside[i[keep], j[keep]] = True
    inside = inside | inside.T
    adj[b[:, None], b[None, :]] = inside
    adj[:, 0] = adj[0, :]
    return adj


def _batch_specs(case):
    # the shapes belong to the case, the edges to the seed
    rng = np.random.default_rng([case["graphs"], 4])
    specs = []
    for _ in range(case["graphs"]):
        k = int(rng.integers(4, 17))
        sizes = [int(s) for s in rng.integers(8, 129, size=k)]
        specs.append((k, sizes, float(rng.uniform(0.2, 0.8)), bool(rng.random() < 0.1)))
    return specs


def _serve_specs(case):
    rng = np.random.default_rng([case["requests"], case["top"], 5])
    specs = []
    for _ in range(case["requests"]):
        n = int(round(math.exp(rng.uniform(math.log(200), math.log(case["top"])))))
        k = int(rng.integers(5, 31))
        specs.append((k, _near_equal(n, k), float(rng.uniform(0.2, 0.9))))
    return specs


def _line(x, q):
    return (x + q - 1) // q * q


def prepare(case, seed):
    kz = _kz()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    kind = case["kind"]
    state = {"case": case}
    if kind == "dense":
        n, k = case["n"], case["k"]
        rng = np.random.default_rng([seed, 1])
        colour = torch.from_numpy(rng.permutation(np.arange(n) % k).astype(np.int32)).cuda()
        adj = _symmetric(n, case["p"], gen) & (colour[:, None] != colour[None, :])
        state.update(adj=adj.to(torch.uint8).contiguous(), colour=colour, k=k)
    elif kind == "rows":
        rows, colour = _rows_graph(_near_equal(case["n"], case["k"]), case["p"], seed, 0, case["plant"])
        state.update(rows=rows, colour=colour, k=case["k"])
        if case["call"] == "async":
            state.update(vmask=torch.zeros(case["n"], dtype=torch.uint8, device="cuda"),
                         emask=torch.zeros_like(rows),
                         out=torch.zeros(kzb.KZ_OUT_BYTES, dtype=torch.uint8, device="cuda"))
    elif kind == "csr":
        row_ptr, col_idx, colour = _sparse(case["n"], case["k"], case["m"], gen)
        state.update(row_ptr=row_ptr, col_idx=col_idx, colour=colour, k=case["k"])
    elif kind == "batch":
        specs = _batch_specs(case)
        b = kzb.Batch.allocate([(sum(s), _words(s), k) for k, s, _, _ in specs], torch.device("cuda", 0))
        if case["less"]:
            b.desc["clique"] = b.desc["k"] - case["less"]
            b.desc_dev = torch.from_numpy(b.desc.view(np.uint8)).cuda()
        rows, colour = b.rows.data_ptr(), b.colour.data_ptr()
        for i, (k, sizes, p, plant) in enumerate(specs):
            _gen(sizes, p, seed, i, plant, rows + 8 * int(b.desc[i]["row_offset"]),
                 colour + 4 * int(b.desc[i]["vertex_offset"]))
        b.vmask.zero_()
        b.emask.zero_()
        state.update(batch=b, run=kzb.BatchKernelizer(kz))
    elif kind == "serve":
        specs = _serve_specs(case)
        reqs, vo, ro = [], 0, 0
        for i, (k, sizes, p) in enumerate(specs):
            rows, colour = _rows_graph(sizes, p, seed, i)
            n, R = rows.shape
            reqs.append((rows, colour, k, vo, ro, n, R))
            vo, ro = _line(vo + n, 128), _line(ro + n * R, 16)
        vmask = torch.zeros(vo, dtype=torch.uint8, device="cuda")
        emask = torch.zeros(ro, dtype=torch.int64, device="cuda")
        state.update(server=_server(), vmask=vmask, emask=emask,
                     requests=[(rows, colour, k, vmask[v:v + n], emask[r:r + n * R].view(n, R))
                               for rows, colour, k, v, r, n, R in reqs])
    elif kind == "dominance":
        state.update(rows=_plain_rows(_dominance_graph(case["n"], gen)))
    elif kind == "clique":
        rows, colour = _rows_graph([case["size"]] * case["k"], case["p"], seed, 0, True)
        state.update(rows=rows, colour=colour, k=case["k"])
    elif kind == "struction":
        state.update(rows=_plain_rows(_struction_graph(case["n"], case["p"], gen)))
    else:
        state.update(rows=_plain_rows(_symmetric(case["n"], case["p"], gen)),
                     priority=torch.randint(-2**62, 2**62, (case["n"],), generator=gen, device="cuda"))
    return state


# ------------------------------------------------------------------ one call
def _numbers(res, names=RESULT):
    return [res[x] for x in names]


def run(state):
    kz = _kz()
    case = state["case"]
    kind = case["kind"]
    if kind == "dense":
        v, e, res = kz.kernelize_dense(state["adj"], state["colour"], state["k"])
        return v, e, _numbers(res)
    if kind == "rows":
        if case["call"] == "async":
            kz.run_async(kzb.graph_bitset(state["rows"]), state["colour"], state["k"], state["vmask"],
                         state["emask"], state["out"], npasses=4)
            return state["vmask"], state["emask"], state["out"]
        v, e, res = kz.kernelize_bitset(state["rows"], state["colour"], state["k"])
        return v, e, _numbers(res)
    if kind == "csr":
        v, e, res = kz.kernelize_csr(state["row_ptr"], state["col_idx"], state["colour"], state["k"])
        return v, e, _numbers(res)
    if kind == "batch":
        b = state["batch"]
        state["run"].run(b)
        return b.vmask, b.emask, b.results
    if kind == "serve":
        return _serve(state)
    if kind == "dominance":
        out = []
        for name, mode in (("vertex", kzb.KZ_DOM_VERTEX), ("edge", kzb.KZ_DOM_EDGE)):
            if case["mode"] in (name, "both"):
                v, e, res = kz.dominance(state["rows"], mode)
                out.append((v, e, _numbers(res, DOM_RESULT)))
        return out
    if kind == "clique":
        # nodes and roots of the result depend on the search's schedule
        clique, res = kz.find_clique(state["rows"], state["colour"], state["k"])
        return clique, res["found"]
    if kind == "struction":
        rows, nodes, res = kz.struction(state["rows"], 0)
        return rows, nodes, _numbers(res, ("nodes", "a_nodes", "c_nodes", "input_edges"))
    colour, res = kz.colour_jp(state["rows"], case["n"], state["priority"])
    return colour, _numbers(res, ("rounds", "colours"))


def _serve(state):
    server = state["server"]
    left = list(enumerate(state["requests"]))[::-1]
    which, results, done = {}, [None] * len(left), 0
    while done < len(results):
        while left:
            i, req = left[-1]
            ticket = server.submit(*req)
            if ticket is None:
                break
            which[ticket] = i
            left.pop()
        for ticket, res in server.done():
            results[which[ticket]] = _numbers(res)
            done += 1
    return state["vmask"], state["emask"], np.array(results, np.int64)


# ------------------------------------------------------------------ necessary work
def _graph_work(sizes, p, fmt_bytes):
    """Bytes of one bit-row graph in and out, and one 64-bit AND and test (four 32-bit
    operations) for every edge and third class."""
    n, k = sum(sizes), len(sizes)
    pairs = (n * n - sum(s * s for s in sizes)) / 2
    return fmt_bytes, pairs * p * max(k - 2, 0) * 4


def work(case):
    kind = case["kind"]
    if kind == "dense":
        n, k = case["n"], case["k"]
        b, f = _graph_work(_near_equal(n, k), case["p"], 2 * n * n + 5 * n)
    elif kind == "rows":
        sizes = _near_equal(case["n"], case["k"])
        b, f = _graph_work(sizes, case["p"], 16 * case["n"] * _words(sizes) + 5 * case["n"])
    elif kind == "csr":
        n, k, m = case["n"], case["k"], case["m"]
        b, f = 8 * n + 8 * m + 2 * m + 5 * n, m * 4
    elif kind in ("batch", "serve"):
        b = f = 0
        specs = _batch_specs(case) if kind == "batch" else _serve_specs(case)
        for s in specs:
            n = sum(s[1])
            gb, gf = _graph_work(s[1], s[2], 16 * n * _words(s[1]) + 5 * n)
            b, f = b + gb, f + gf
    elif kind == "dominance":
        n = case["n"]
        b = 16 * n * ((n + 63) // 64) + n
        b, f = b * (2 if case["mode"] == "both" else 1), n * n / 2
    elif kind == "clique":
        sizes = [case["size"]] * case["k"]
        b, f = 8 * sum(sizes) * _words(sizes), sum(sizes) * _words(sizes) * 2
    elif kind == "struction":
        n, p = case["n"], case["p"]
        nodes = n * p + (n * (1 - p)) ** 2 / 2 * p
        b, f = nodes * nodes / 8 + 8 * nodes + n * n / 8, nodes * nodes / 64
    else:
        n = case["n"]
        b, f = n * n / 8 + 12 * n, n * n / 2 * case["p"] * 2
    return {"bytes": float(b), "flops": float(f)}


def exact(case, seed):
    # every output is a whole number or a bit mask, compared bit for bit: none is a rounded value
    return None
