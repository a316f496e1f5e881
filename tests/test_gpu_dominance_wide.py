"""Dominance of rows wider than a wave: every number of words a lane holds, with
nodes in all of them.  Few edges among many nodes against the definitions on sets
(the nodes without an edge go in the first step), and dense graphs with twins and
nodes inside others, which are the only ones to go (a product of the adjacency
with its complement counts who is inside whom).  And a star's edges go in a few
times what its nodes take (every leaf looked at every other one before)."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2212_00574_amd.binding import KZ_DOM_EDGE, KZ_DOM_VERTEX, Kernelizer  # noqa: E402


def vertex_sets(n, nbr):
    alive, steps, sweeps, edges = set(range(n)), 0, 0, 0
    nbr = {v: set(s) for v, s in nbr.items()}
    none = set()
    while True:
        any_gone = False
        for b in range(n):
            if b not in alive:
                continue
            nb = nbr.get(b, none)
            gone = [a for a in alive if a != b and a not in nb and nbr.get(a, none) <= nb]
            if gone:
                steps += 1
                any_gone = True
                for a in gone:
                    edges += len(nbr.get(a, none))
                    for u in nbr.pop(a, none):
                        nbr[u].discard(a)
                alive -= set(gone)
        if not any_gone:
            return alive, nbr, sweeps, steps, edges
        sweeps += 1


def edge_sets(nbr):
    nbr = {v: set(s) for v, s in nbr.items()}
    sweeps = deleted = 0
    while True:
        any_gone = False
        for a in sorted(nbr):
            for u in sorted(nbr[a]):
                both = nbr[a] & nbr[u]
                if any(b != a and b not in nbr[a] and both <= nbr[b] for b in nbr[u]):
                    nbr[a].discard(u)
                    nbr[u].discard(a)
                    deleted += 1
                    any_gone = True
        if not any_gone:
            return nbr, sweeps, deleted
        sweeps += 1


def pack(n, R, nbr):
    rows = np.zeros((n, R), np.uint64)
    for v, s in nbr.items():
        for u in s:
            rows[v, u >> 6] |= np.uint64(1) << np.uint64(u & 63)
    return rows


@pytest.mark.parametrize("n,R", [(64, 1), (65, 2), (128, 2), (2049, 33), (4096, 64), (4097, 65), (9000, 200), (16385, 257),
                                 (30000, 512), (33000, 516)])
def test_few_edges_in_wide_rows(n, R):
    rng = np.random.default_rng(n)
    some = rng.choice(n, min(n, 70), replace=False)
    nbr = {int(v): set() for v in some}

    def join(a, b):
        if a != b:
            nbr[int(a)].add(int(b))
            nbr[int(b)].add(int(a))

    for a, b in rng.choice(some, (260, 2)):
        join(a, b)
    for v in some[2:40]:  # nodes next to most, and to each other
        join(some[0], v)
        join(some[1], v)
    rows = torch.from_numpy(pack(n, R, nbr).view(np.int64)).cuda()
    kz = Kernelizer(0)
    try:
        print("dominance wide", n, R, flush=True)
        vm, em, res = kz.dominance(rows, KZ_DOM_VERTEX)
        alive, left, sweeps, steps, edges = vertex_sets(n, nbr)
        assert np.array_equal(np.flatnonzero(vm.cpu().numpy()), sorted(alive))
        assert np.array_equal(em.cpu().numpy().view(np.uint64), pack(n, R, left))
        assert (res["sweeps"], res["events"], res["deleted_edges"]) == (sweeps, steps, edges)
        vm, em, res = kz.dominance(rows, KZ_DOM_EDGE)
        left, sweeps, deleted = edge_sets(nbr)
        assert np.array_equal(em.cpu().numpy().view(np.uint64), pack(n, R, left))
        assert (res["sweeps"], res["deleted_edges"]) == (sweeps, deleted)
    finally:
        kz.close()


@pytest.mark.parametrize("n,p", [(2049, 0.3), (4096, 0.02), (4500, 0.4), (9000, 0.1), (16500, 0.3), (33000, 0.3)])
def test_dense_graphs_lose_their_twins(n, p):
    gen = torch.Generator(device="cuda").manual_seed(n)
    a = torch.triu(torch.rand((n, n), generator=gen, device="cuda") < p, 1)
    a = a | a.T
    rng = np.random.default_rng(n)
    pick = rng.permutation(n)
    ends = torch.from_numpy(pick[:24].copy()).cuda()
    for i in range(12):  # a twin, or a node inside another: no edges among these, so that none waits for another
        keep, other = int(pick[2 * i]), int(pick[2 * i + 1])
        a[keep, ends] = False
        a[ends, keep] = False
        row = a[keep].clone()
        row[ends] = False
        if i % 2:
            row &= torch.rand(n, generator=gen, device="cuda") < 0.7
        a[other, :] = row
        a[:, other] = row
    words = (n + 63) // 64
    bits = torch.zeros((n, words * 64), dtype=torch.bool, device="cuda")
    bits[:, :n] = a
    rows = torch.empty((n, words * 8), dtype=torch.uint8, device="cuda")
    shift = torch.arange(8, device="cuda", dtype=torch.uint8)
    for i in range(0, n, 2048):
        rows[i:i + 2048] = (bits[i:i + 2048].view(-1, words * 8, 8).to(torch.uint8) << shift).sum(2, dtype=torch.uint8)
    rows = rows.view(torch.int64)
    alive = torch.ones(n, dtype=torch.bool, device="cuda")
    steps = sweeps = 0
    while True:  # sweeps over the pairs that a product finds
        f = (a & alive[None, :]).to(torch.float32)
        pairs = []
        for i in range(0, n, 4096):
            outside = f[i:i + 4096] @ (1 - f).T  # [a, b]: neighbours of a that b lacks (b itself among them if adjacent)
            inside = (outside == 0) & alive[i:i + 4096, None] & alive[None, :]
            inside[torch.arange(inside.shape[0], device="cuda"), torch.arange(i, i + inside.shape[0], device="cuda")] = False
            pairs += [(int(y), i + int(x)) for x, y in inside.nonzero().cpu().numpy()]
        if not pairs:
            break
        sweeps += 1
        gone = set()
        for b in sorted({b for b, _ in pairs}):
            mine = [x for y, x in pairs if y == b and x not in gone] if b not in gone else []
            steps += bool(mine)
            gone |= set(mine)
        alive[list(gone)] = False
    kz = Kernelizer(0)
    try:
        print("dominance twins", n, p, int(n - alive.sum()), flush=True)
        vm, em, res = kz.dominance(rows, KZ_DOM_VERTEX)
        assert torch.equal(vm.bool(), alive)
        keep = torch.zeros(words * 64, dtype=torch.bool, device="cuda")
        keep[:n] = alive
        mask = (keep.view(words * 8, 8).to(torch.uint8) << shift).sum(1, dtype=torch.uint8).view(torch.int64)
        assert torch.equal(em, torch.where(alive[:, None], rows & mask, torch.zeros_like(rows)))
        assert (res["sweeps"], res["events"]) == (sweeps, steps)
    finally:
        kz.close()


@pytest.mark.parametrize("n", [2049, 4097, 17000])
def test_a_step_deletes_nearly_all(n):
    """Nodes all next to the same three: the first takes all the others, with their
    edges, and of the three the first then takes the others."""
    R = (n + 63) // 64
    hubs = (5, 70, n - 1)
    nbr = {v: set(hubs) for v in range(n) if v not in hubs}
    nbr.update({h: set(nbr) - set(hubs) for h in hubs})
    kz = Kernelizer(0)
    try:
        print("dominance nearly all", n, flush=True)
        vm, em, res = kz.dominance(torch.from_numpy(pack(n, R, nbr).view(np.int64)).cuda(), KZ_DOM_VERTEX)
        assert np.flatnonzero(vm.cpu().numpy()).tolist() == [0, 5]
        assert np.array_equal(em.cpu().numpy().view(np.uint64), pack(n, R, {0: {5}, 5: {0}}))
        assert (res["sweeps"], res["events"], res["deleted_edges"]) == (1, 2, 3 * (n - 4) + 2)
    finally:
        kz.close()


def test_a_star_takes_few_turns():
    n = 2100
    nbr = {0: set(range(1, n)), **{v: {0} for v in range(1, n)}}
    rows = torch.from_numpy(pack(n, 33, nbr).view(np.int64)).cuda()
    rng = np.random.default_rng(1)
    adj = np.triu(rng.random((n, n)) < 0.9, 1)
    adj |= adj.T
    full = torch.from_numpy(np.packbits(np.pad(adj, ((0, 0), (0, 33 * 64 - n))), axis=1, bitorder="little").view(np.int64)).cuda()
    kz = Kernelizer(0)
    try:
        took = []
        for r in (rows, full):
            best = 1e9
            for _ in range(3):
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                kz.dominance(r, KZ_DOM_EDGE)
                torch.cuda.synchronize()
                best = min(best, time.perf_counter() - t0)
            took.append(best)
        assert took[0] < took[1], took  # two sweeps of short steps; a dense graph's took less than the star's
    finally:
        kz.close()
