"""The colouring's two ways, by rounds and by blocks of 64 vertices: dense graphs
whose priorities leave them few rounds (the sides of a bipartite graph one after
the other, classes in order, hubs first), many rounds, and a few rounds behind
many, against the greedy colouring in order of falling keys; a malformed graph is
refused before its first round; and few rounds cost the time of few rounds (by
blocks they took thirty times as long)."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2212_00574_amd import inputs  # noqa: E402
from paper_2212_00574_amd.binding import Kernelizer  # noqa: E402


def greedy(adj, pri):
    n = len(adj)
    order = sorted(range(n), key=lambda v: (int(pri[v]), v), reverse=True)
    colour, level = np.full(n, -1, np.int64), np.zeros(n, np.int64)
    for v in order:
        before = np.flatnonzero(adj[v] & (colour >= 0))
        free = np.ones(len(before) + 1, bool)
        held = colour[before]
        free[held[held < len(free)]] = False
        colour[v] = np.argmax(free)
        level[v] = 1 + (level[before].max() if len(before) else 0)
    return colour, int(level.max())


def graph(kind, n, rng):
    side = np.arange(n) * (int(kind[1:]) if kind[0] == "k" else 2) // n
    if kind[0] == "k":  # complete between classes
        a = side[:, None] != side[None, :]
    elif kind[0] == "h":  # hubs next to all others, and to each other
        a = np.zeros((n, n), bool)
        a[:int(kind[1:])] = True
        a |= a.T
    elif kind[0] == "u":  # a few vertices next to all of a complete bipartite graph
        a = side[:, None] != side[None, :]
        a[:int(kind[1:])] = True
        a |= a.T
    else:
        a = np.triu(rng.random((n, n)) < float(kind[1:]), 1)
        a |= a.T
    np.fill_diagonal(a, False)
    return a


@pytest.mark.parametrize("n", [511, 512, 1100, 2500])
@pytest.mark.parametrize("kind", ["k2", "k7", "k40", "h12", "u6", "u30", "p0.02", "p0.4"])
def test_ways_match_greedy(kind, n):
    rng = np.random.default_rng(n)
    adj = graph(kind, n, rng)
    rows = torch.from_numpy(inputs.dense_to_rows(adj.astype(np.uint8)).view(np.int64)).cuda()
    kz = Kernelizer(0)
    try:
        for name, pri in (("falling", np.arange(n, 0, -1)), ("equal", np.zeros(n)), ("random", rng.integers(0, 2**63, n))):
            print("colouring ways", kind, n, name, flush=True)
            pri = pri.astype(np.uint64)
            col, res = kz.colour_jp(rows, n, torch.from_numpy(pri.view(np.int64)).cuda())
            want, rounds = greedy(adj, pri)
            assert np.array_equal(col.cpu().numpy(), want), (kind, n, name)
            assert res["rounds"] == rounds and res["colours"] == int(want.max()) + 1
    finally:
        kz.close()


def test_refused_before_a_round():
    n = 1000
    adj = graph("p0.3", n, np.random.default_rng(1)).astype(np.uint8)
    pri = torch.arange(n, device="cuda")
    kz = Kernelizer(0)
    try:
        for spoil, status in (((5, 900), -4), ((7, 7), -5)):
            bad = adj.copy()
            bad[spoil] ^= 1
            rows = torch.from_numpy(inputs.dense_to_rows(bad).view(np.int64)).cuda()
            col, res = kz.colour_jp(rows, n, pri, check=False)
            assert res["status"] == status
    finally:
        kz.close()


def test_few_rounds_take_their_time():
    n = 8192
    side = torch.arange(n, device="cuda") * 2 // n
    half = torch.zeros((n, n // 64), dtype=torch.int64, device="cuda")
    half[:n // 2, n // 128:] = -1
    half[n // 2:, :n // 128] = -1
    falling = torch.arange(n, 0, -1, device="cuda")
    mixed = torch.randperm(n, generator=torch.Generator(device="cuda").manual_seed(2), device="cuda")
    kz = Kernelizer(0)
    try:
        took = []
        for pri in (falling, mixed):
            best = 1e9
            for _ in range(4):
                t0 = time.perf_counter()
                col, res = kz.colour_jp(half, n, pri)
                torch.cuda.synchronize()
                best = min(best, time.perf_counter() - t0)
            took.append(best)
            if pri is falling:
                assert res["rounds"] == 2 and torch.equal(col, side.to(torch.int32))
            else:
                assert res["rounds"] > 1000 and res["colours"] == 2
        assert 3 * took[0] < took[1], took  # 2 rounds, thousands of them
    finally:
        kz.close()
