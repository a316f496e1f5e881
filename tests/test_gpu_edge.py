"""The edge test's matrix product and its per-lane search against the oracle, bit for bit, at the sizes where
they split: block and class-chunk edges, odd block counts, searches that run to a row's last word, more edges
left than a wave lists at once, and the squared tile order."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle import kernelize_bitset  # noqa: E402
from paper_2212_00574_amd import inputs  # noqa: E402
from paper_2212_00574_amd.binding import Kernelizer  # noqa: E402

from test_gpu_parity import check_same, run_bitset  # noqa: E402

CASES = {
    "blocks": ([1, 63, 64, 65, 127, 128, 129], 0.6),
    "odd block count": ([64, 65, 128, 129, 30], 0.4),
    "one vertex each": ([1] * 9, 0.9),
    "empty class": ([70, 0, 70, 70], 0.6),
    "two classes": ([130, 70], 0.3),
    "chunk 12": ([40] * 12, 0.8),
    "chunk 13": ([40] * 13, 0.8),
    "chunk 20": ([33] * 20, 0.85),
    "chunk 21": ([33] * 21, 0.85),
    "chunk 32": ([20] * 32, 0.9),
    "chunk 33": ([20] * 33, 0.9),
    "chunks 65": ([10] * 65, 0.95),
    "squares": ([2] * 190, 0.97),
    "long search": ([700, 699, 641, 640], 0.06),
    "lists": ([128] * 4, 0.36),
    "product skipped": ([200] * 16, 0.12),
}


@pytest.mark.parametrize("name", list(CASES))
def test_edge_sizes(name):
    sizes, p = CASES[name]
    kz = Kernelizer(0)
    for seed in (0, 1):
        rows, colour, _ = inputs.make_graph(sizes, p, seed=seed, gid=7, plant=0 not in sizes and seed == 1).bitset()
        res, vm, em = run_bitset(kz, rows, colour, len(sizes), "%s/%d" % (name, seed))
        check_same(res, kernelize_bitset(rows, colour, len(sizes)), vm, em, name)
    kz.close()
