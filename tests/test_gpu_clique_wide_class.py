"""kz_find_clique where class 0 is large: the counts of its vertices' roots are
summed up by one workgroup, 4096 a turn, around the ends of its waves' quarters and
turns; the smallest clique is the only one, or the first of two."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2212_00574_amd.binding import Kernelizer  # noqa: E402


@pytest.mark.parametrize("s0", [1, 4, 255, 4095, 4096, 4097, 16384, 20001])
def test_large_class_zero(s0):
    rng = np.random.default_rng(s0)
    sizes = [s0, 70, 3]
    start, words = np.cumsum([0] + sizes), [(s + 63) // 64 for s in sizes]
    first = np.cumsum([0] + words)
    n, R = int(start[-1]), int(first[-1])
    rows = np.zeros((n, R), np.uint64)

    def join(a, b):
        for u, v in ((a, b), (b, a)):
            c = int(np.searchsorted(start, v, side="right")) - 1
            j = v - int(start[c])
            rows[u, first[c] + j // 64] |= np.uint64(1) << np.uint64(j % 64)

    # pairs of classes 0 and 1 without a third vertex, then the cliques
    for v in rng.choice(s0, min(s0, 900), replace=False):
        join(int(v), s0 + int(rng.integers(0, 70)))
    at = sorted({int(x) for x in rng.integers(0, s0, 2)})
    cliques = [(v, s0 + int(rng.integers(0, 70)), s0 + 70 + int(rng.integers(0, 3))) for v in at]
    for v, a, b in cliques:
        join(v, a)
        join(v, b)
        join(a, b)
    colour = np.repeat(np.arange(3), sizes).astype(np.int32)
    kz = Kernelizer(0)
    try:
        r, c = torch.from_numpy(rows.view(np.int64)).cuda(), torch.from_numpy(colour).cuda()
        for dead in (None, at[0]):
            vm = None
            if dead is not None:
                vm = torch.ones(n, dtype=torch.uint8, device="cuda")
                vm[dead] = 0
            print("clique class 0", s0, dead, flush=True)
            got, res = kz.find_clique(r, c, 3, vm)
            # by definition: v0 and its neighbours in class 1, then a common one in class 2
            want = None
            for v in range(s0):
                if want or v == dead:
                    continue
                for j in range(70):
                    if not (rows[v, first[1] + j // 64] >> np.uint64(j % 64)) & np.uint64(1):
                        continue
                    both = int(rows[v, first[2]] & rows[s0 + j, first[2]])
                    if both:
                        want = [v, s0 + j, s0 + 70 + (both & -both).bit_length() - 1]
                        break
            assert res["found"] == (want is not None)
            assert got.cpu().numpy().tolist() == (want or [-1, -1, -1]), (s0, dead)
    finally:
        kz.close()
