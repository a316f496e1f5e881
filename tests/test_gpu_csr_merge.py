"""The sparse edge test where lanes merge rows by themselves, against the oracle:
rows of a few entries (grids, rings, trees, the smallest graphs), rows that begin
alike (cliques, hubs, with few and many classes to find), such rows that part again
soon after, and both kinds beside longer rows; found, failed and over several
rounds.  And cliques cost less than random rows of as many entries (0.16 of their time; 0.43
when every row was searched by its wave)."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle import kernelize_csr  # noqa: E402
from paper_2212_00574_amd.binding import Kernelizer  # noqa: E402

from test_gpu_parity import check_same, run_csr  # noqa: E402


def csr(n, pairs, colour):
    a, b = np.asarray(pairs, np.int64).reshape(-1, 2).T
    keep = colour[a] != colour[b]
    key = np.unique(np.concatenate([a[keep] * n + b[keep], b[keep] * n + a[keep]]))
    rp = np.zeros(n + 1, np.int64)
    rp[1:] = np.cumsum(np.bincount(key // n, minlength=n))
    return rp, (key % n).astype(np.int32)


def grid(w, holes, rng):
    x, y = np.meshgrid(np.arange(w), np.arange(w))
    i = (y * w + x).ravel()
    x, y = x.ravel(), y.ravel()
    p = np.concatenate([np.stack([i[x < w - 1], i[x < w - 1] + 1], 1), np.stack([i[y < w - 1], i[y < w - 1] + w], 1),
                        np.stack([i[(x < w - 1) & (y < w - 1)], i[(x < w - 1) & (y < w - 1)] + w + 1], 1)])
    return w * w, p[rng.random(len(p)) >= holes], ((x + y) % 3).astype(np.int32)


def cliques(n, size, k, rng, parted=0):
    c = np.arange(n)
    p = np.concatenate([np.stack([c, c // size * size + (c + d) % size], 1) for d in range(1, size)])
    if parted:  # an early neighbour for all, then rows of their own
        p = np.concatenate([p[rng.random(len(p)) < 0.3]] + [np.stack([c, np.full(n, h)], 1) for h in range(parted)])
    return n, p, (c % k).astype(np.int32)


def ring(n, w, k, rng, far=0.2):
    q = np.tile(np.arange(n), w)
    o = (q + np.repeat(np.arange(1, w + 1), n)) % n
    o = np.where(rng.random(len(o)) < far, rng.integers(0, n, len(o)), o)
    return n, np.stack([q, o], 1), rng.integers(0, k, n).astype(np.int32)


def hubs(n, h, d, k, rng):
    p = np.concatenate([np.stack([np.tile(np.arange(n), h), np.repeat(np.arange(h), n)], 1), rng.integers(0, n, (n * d, 2))])
    return n, p, rng.integers(0, k, n).astype(np.int32)


CASES = {
    "grid": lambda r: grid(37, 0.0, r), "grid with holes": lambda r: grid(41, 0.1, r),
    "triangle": lambda r: (3, [(0, 1), (1, 2), (0, 2)], np.arange(3, dtype=np.int32)),
    "two edges": lambda r: (3, [(0, 1), (1, 2)], np.arange(3, dtype=np.int32)),
    "one edge": lambda r: (2, [(0, 1)], np.arange(2, dtype=np.int32)),
    "tree": lambda r: (500, np.stack([np.arange(1, 500), np.arange(1, 500) // 3], 1), (np.arange(500) % 3).astype(np.int32)),
    "ring 6": lambda r: ring(1500, 6, 3, r), "ring 12": lambda r: ring(900, 12, 4, r), "ring 20": lambda r: ring(700, 20, 5, r),
    "ring 30 of 8": lambda r: ring(600, 30, 8, r, 0.05),
    "cliques 3": lambda r: cliques(1200, 60, 3, r), "cliques 5": lambda r: cliques(1000, 50, 5, r),
    "cliques 8": lambda r: cliques(900, 90, 8, r), "cliques 9": lambda r: cliques(900, 90, 9, r),
    "cliques 70": lambda r: cliques(840, 280, 70, r), "cliques 300": lambda r: cliques(700, 350, 300, r),
    "parted 3": lambda r: cliques(900, 30, 3, r, 1), "parted 4": lambda r: cliques(900, 30, 4, r, 2),
    "parted 8": lambda r: cliques(900, 45, 8, r, 4),
    "hubs": lambda r: hubs(1500, 4, 3, 3, r), "hubs 4": lambda r: hubs(1200, 12, 10, 4, r), "hubs 5": lambda r: hubs(1200, 40, 15, 5, r),
}


@pytest.mark.parametrize("name", list(CASES))
def test_lanes_merge(name):
    kz = Kernelizer(0)
    try:
        for seed in (0, 1):
            rng = np.random.default_rng(seed)
            n, pairs, colour = CASES[name](rng)
            if seed:  # other places in the rows
                perm = rng.permutation(n)
                pairs, col = perm[np.asarray(pairs)], np.empty_like(colour)
                col[perm] = colour
                colour = col
            k = int(colour.max()) + 1
            rp, ci = csr(n, pairs, colour)
            print("csr merge", name, seed, n, len(ci), flush=True)
            res, vm, em = run_csr(kz, rp, ci, colour, k, "%s/%d" % (name, seed))
            check_same(res, kernelize_csr(rp, ci, colour, k), vm, em, name)
    finally:
        kz.close()


def test_cliques_cost_less_than_random_rows():
    n, size, k = 40000, 200, 3
    c = torch.arange(n, device="cuda")
    colour = (c % k).to(torch.int32)
    gen = torch.Generator(device="cuda").manual_seed(3)

    def entries(a, b):
        keep = colour[a] != colour[b]
        key = torch.unique(torch.cat([a[keep] * n + b[keep], b[keep] * n + a[keep]]))
        rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
        rp[1:] = torch.cumsum(torch.bincount(key // n, minlength=n), 0)
        return rp, (key % n).to(torch.int32)

    graphs = [entries(c.repeat_interleave(size), (c // size * size).repeat_interleave(size) +
                      torch.arange(size, device="cuda").repeat(n))]
    m = graphs[0][1].numel() * 3 // 4
    graphs.append(entries(torch.randint(0, n, (m,), generator=gen, device="cuda"),
                          torch.randint(0, n, (m,), generator=gen, device="cuda")))
    kz = Kernelizer(0)
    try:
        took = []
        for rp, ci in graphs:
            best = 1e9
            for _ in range(6):
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                kz.kernelize_csr(rp, ci, colour, k)
                torch.cuda.synchronize()
                best = min(best, time.perf_counter() - t0)
            took.append(best / ci.numel())
        assert took[0] < 0.3 * took[1], took
    finally:
        kz.close()
