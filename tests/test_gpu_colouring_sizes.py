"""The colouring where its one workgroup changes what it keeps in LDS: vertices beyond 16384, colours beyond 2047
(bitmaps in memory), the ends of the 64-vertex blocks, and sparse graphs, which run the rounds themselves.  The colours are those of the greedy
colouring in order of falling keys, each vertex one round after the last neighbour before it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2212_00574_amd.binding import Kernelizer  # noqa: E402


def greedy(n, nbrs, pri):
    order = sorted(range(n), key=lambda v: (int(pri[v]), v), reverse=True)
    colour, level = np.full(n, -1, np.int64), np.zeros(n, np.int64)
    for v in order:
        before = nbrs[v][colour[nbrs[v]] >= 0]
        free = np.ones(len(before) + 1, bool)
        held = colour[before]
        free[held[held < len(free)]] = False
        colour[v] = np.argmax(free)
        level[v] = 1 + (level[before].max() if len(before) else 0)
    return colour, int(level.max())


@pytest.mark.parametrize("n,degree,hubs,clique", [(64, 10, 0, 40), (127, 20, 0, 90), (129, 30, 1, 129), (1000, 40, 2, 300),
                                                  (4097, 12, 1, 200), (4300, 12, 3, 70), (16384, 8, 0, 80),
                                                  (16385, 8, 0, 150), (16500, 8, 2, 90), (3000, 40, 0, 60), (16500, 200, 1, 90), (4300, 12, 0, 2200)])
def test_colouring_sizes(n, degree, hubs, clique):
    """Random edges, `hubs` vertices next to all others, and a clique of the wanted size."""
    rng = np.random.default_rng(n)
    u, v = rng.integers(0, n, (2, n * degree // 2))
    pairs = [(u, v)] + [(np.full(n, h), np.arange(n)) for h in range(hubs)]
    members = rng.choice(n, clique, replace=False)
    pairs.append((np.repeat(members, clique), np.tile(members, clique)))
    u, v = np.concatenate([p[0] for p in pairs]), np.concatenate([p[1] for p in pairs])
    keep = u != v
    u, v = np.concatenate([u[keep], v[keep]]), np.concatenate([v[keep], u[keep]])
    rows = np.zeros((n, (n + 63) // 64), np.uint64)
    np.bitwise_or.at(rows, (u, v >> 6), np.uint64(1) << (v & 63).astype(np.uint64))
    key = np.unique(u * n + v)
    nbrs = np.split(key % n, np.searchsorted(key // n, np.arange(1, n)))
    pri = rng.integers(0, 2**64, n, dtype=np.uint64)
    pri[::7] = pri[0]  # equal priorities: the index decides
    print("colouring sizes", n, degree, hubs, clique, flush=True)
    kz = Kernelizer(0)
    col, res = kz.colour_jp(torch.from_numpy(rows.view(np.int64)).cuda(), n, torch.from_numpy(pri.view(np.int64)).cuda())
    torch.cuda.synchronize()
    want, rounds = greedy(n, nbrs, pri)
    assert np.array_equal(col.cpu().numpy(), want), n
    assert res["rounds"] == rounds and res["colours"] == int(want.max()) + 1
    kz.close()
