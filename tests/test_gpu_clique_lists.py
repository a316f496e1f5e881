"""kz_find_clique against the oracle where the search by lists splits: fewer
and more roots than waves, classes over one and over 64 words (the roots are
found 64 class-0 vertices and 64 class-1 words at a time), lists that fill
their room, picks whose rest is wider than a wave, lists in LDS and in the workspace, dead vertices in classes 0
and 1, k = 1 to 4."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle import find_clique  # noqa: E402
from paper_2212_00574_amd import inputs  # noqa: E402
from paper_2212_00574_amd.binding import Kernelizer  # noqa: E402

DEV = torch.device("cuda", 0)

CASES = [  # class sizes, p, plant, share of live vertices
    ([1], 0.0, False, 1.0), ([70], 0.0, False, 0.02), ([3, 65], 0.02, True, 1.0), ([200, 300], 0.0005, False, 0.9),
    ([64, 64, 64], 0.02, True, 1.0), ([65, 1, 129], 0.05, False, 1.0), ([4200, 3, 40], 0.01, True, 0.5),
    ([2, 4200, 30, 5], 0.01, True, 1.0), ([63, 65, 64, 66], 0.05, True, 0.8), ([90] * 12, 0.35, False, 1.0),
    ([90] * 12, 0.35, True, 0.9), ([33] * 20, 0.6, False, 1.0), ([20] * 8, 1.0, False, 0.5),
    ([1] * 64, 1.0, False, 1.0), ([2] * 64, 0.9, True, 1.0), ([10, 10, 10, 1500, 1500, 1500], 0.02, False, 1.0),
    ([10, 10, 10, 1500, 1500, 1500], 0.1, True, 1.0), ([1, 1, 300, 64, 64, 64, 64, 64], 0.4, False, 1.0),
    ([5, 5, 90, 4200, 40, 4100], 0.2, False, 0.7), ([40] * 6, 0.0, False, 1.0), ([450] * 20, 0.05, True, 1.0),
]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_lists_match_oracle(i):
    sizes, p, plant, live = CASES[i]
    k = len(sizes)
    g = inputs.make_graph(sizes, p, seed=31, gid=i, plant=plant, shuffle=False)
    rows, colour, lay = g.bitset()
    adj = inputs.unpack_rows(rows, lay).astype(np.uint8)
    rng = np.random.default_rng(100 + i)
    vmask = (rng.random(lay.n) < live).astype(np.uint8) if live < 1 else None
    ref, _ = find_clique(adj, colour, k, vmask)
    kz = Kernelizer(0)
    try:
        r = torch.from_numpy(np.ascontiguousarray(rows).view(np.int64)).to(DEV)
        c = torch.from_numpy(np.ascontiguousarray(colour, np.int32)).to(DEV)
        got, res = kz.find_clique(r, c, k, None if vmask is None else torch.from_numpy(vmask).to(DEV))
        torch.cuda.synchronize()
        assert res["found"] == (ref is not None), (res, ref)
        assert got.cpu().numpy().tolist() == ([-1] * k if ref is None else ref.tolist())
        if ref is None:  # every pair was handed out, and every live pick of the first two classes counted
            assert res["roots"] == sizes[0] * (sizes[1] if k > 1 else 1)
    finally:
        kz.close()
