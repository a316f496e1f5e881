"""The reverse entry of every CSR entry is looked for first where it would lie
in an evenly filled row: rows short and long, even, crowded at either end and
with gaps, col_idx aligned and not, are accepted as they are, and refused
(KZ_EASYM) when one reverse entry is swapped for another vertex, wherever it
lies in its row."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2212_00574_amd.binding import Kernelizer  # noqa: E402

DEV = torch.device("cuda", 0)
N, K = 600, 3


def ends(kind, rng):
    """The neighbours of the hub: vertices of other classes than its own."""
    other = np.array([v for v in range(1, N) if v % K != 0])
    if kind == "even":
        return other[::3]
    if kind == "low":
        return other[:70]
    if kind == "high":
        return other[-70:]
    if kind == "gap":
        return np.concatenate([other[:40], other[-9:]])
    if kind == "short":
        return rng.choice(other, 5, replace=False)
    return rng.choice(other, 200, replace=False)


def csr(adj):
    ci = [np.flatnonzero(r) for r in adj]
    rp = np.concatenate([[0], np.cumsum([len(c) for c in ci])]).astype(np.int64)
    return rp, np.concatenate(ci).astype(np.int32)


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("kind", ["even", "low", "high", "gap", "short", "random"])
def test_reverse_entries(kind, shift):
    rng = np.random.default_rng(3)
    adj = np.zeros((N, N), np.uint8)
    hub = 0 if kind in ("even", "low") else N - N % K - K * 20  # a vertex of class 0, low and high
    nb = np.array([v for v in ends(kind, rng) if v != hub])
    adj[hub, nb] = adj[nb, hub] = 1
    extra = rng.integers(0, N, size=(900, 2))
    for u, v in extra:
        if u % K != v % K and hub not in (u, v):
            adj[u, v] = adj[v, u] = 1
    colour = torch.from_numpy((np.arange(N) % K).astype(np.int32)).to(DEV)
    kz = Kernelizer(0)

    def status(a):
        rp, ci = csr(a)
        buf = torch.zeros(len(ci) + shift, dtype=torch.int32, device=DEV)
        buf[shift:] = torch.from_numpy(ci).to(DEV)
        _, _, res = kz.kernelize_csr(torch.from_numpy(rp).to(DEV), buf[shift:], colour, K, check=False)
        return res["status"]

    try:
        assert status(adj) == 0
        for v in rng.permutation(nb)[:12]:
            bad = adj.copy()
            # the hub's entry v becomes another vertex of a class not its own: as many entries as before
            free = [x for x in range(N) if x % K and x != hub and not bad[hub, x]]
            bad[hub, v] = 0
            bad[hub, rng.choice(free)] = 1
            assert status(bad) == -4, (kind, int(v))
            bad = adj.copy()
            bad[v, hub] = 0  # one entry less
            assert status(bad) == -4, (kind, int(v))
    finally:
        kz.close()
