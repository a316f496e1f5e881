"""Struction of rows wider than a wave's 64 words: G' by its definition, what is
wrong with a row found in any of its words, and sparse rows checked in a few times
what reading them takes (a lane per bit of every word took nine times as long)."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2212_00574_amd.binding import Kernelizer, KzError  # noqa: E402


def rows_of(n, R, edges):
    rows = np.zeros((n, R), np.uint64)
    for a, b in edges:
        rows[a, b >> 6] |= np.uint64(1) << np.uint64(b & 63)
        rows[b, a >> 6] |= np.uint64(1) << np.uint64(a & 63)
    return rows


@pytest.mark.parametrize("n,extra", [(4096, 0), (4097, 0), (4160, 3), (8200, 0)])
def test_wide_rows(n, extra):
    rng = np.random.default_rng(n)
    R = (n + 63) // 64 + extra
    pick = rng.integers(0, n, (400, 2))
    edges = {(int(min(a, b)), int(max(a, b))) for a, b in pick if a != b}
    pivot = n - 3
    edges |= {(int(v), pivot) for v in rng.choice(n - 4, 70, replace=False)}
    rows = rows_of(n, R, edges)
    kz = Kernelizer(0)
    try:
        print("struction wide", n, R, flush=True)
        out, mp, res = kz.struction(torch.from_numpy(rows.view(np.int64)).cuda(), pivot)
        near = {a + b - pivot for a, b in edges if pivot in (a, b)}
        inside = sorted(e for e in edges if not (set(e) & near) and pivot not in e)
        nodes = [(v, -1) for v in sorted(near)] + inside
        assert mp.cpu().numpy().tolist() == [list(x) for x in nodes]
        adj = {(a, b) for a, b in edges} | {(b, a) for a, b in edges}
        bits = np.unpackbits(out.cpu().numpy().view(np.uint8), axis=1, bitorder="little")[:, :len(nodes)]
        for i, (x, y) in enumerate(nodes):
            for j, (p, q) in enumerate(nodes):
                if y < 0 and q < 0:
                    want = (x, p) in adj
                elif y < 0:
                    want = (x, p) in adj and (x, q) in adj
                elif q < 0:
                    want = (x, p) in adj and (y, p) in adj
                else:
                    want = x == p and (y, q) in adj
                assert bits[i, j] == want, (i, j)
        for at in (1, n - 2):
            for what, status in (("loop", -5), ("one way", -4), ("past", -1)):
                bad = rows.copy()
                if what == "loop":
                    bad[at, at >> 6] ^= np.uint64(1) << np.uint64(at & 63)
                elif what == "one way":
                    bad[at, (n - 1) >> 6] ^= np.uint64(1) << np.uint64((n - 1) & 63)
                elif R * 64 > n:
                    bad[at, R - 1] ^= np.uint64(1) << np.uint64(63)
                else:
                    continue
                with pytest.raises(KzError) as e:
                    kz.struction(torch.from_numpy(bad.view(np.int64)).cuda(), pivot)
                assert e.value.status == status, (at, what)
    finally:
        kz.close()


def test_sparse_rows_at_the_rate_of_a_copy():
    n = 40000
    R = n // 64
    rows = torch.zeros((n, R), dtype=torch.int64, device="cuda")
    for a, b in ((0, 3), (5, 39999), (77, 20000)):
        rows[a, b >> 6] |= 1 << (b & 63) if (b & 63) < 63 else -2**63
        rows[b, a >> 6] |= 1 << (a & 63)
    other = torch.empty_like(rows)
    kz = Kernelizer(0)

    def best(f):
        t = []
        for _ in range(5):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            f()
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        return min(t)

    try:
        copy, call = best(lambda: other.copy_(rows)), best(lambda: kz.struction(rows, 0))
        assert call < 10 * copy, (call, copy)
    finally:
        kz.close()
