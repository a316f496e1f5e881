"""The sparse edge test's search against the oracle: rows beyond its table, one, four and sixteen words of classes, the
entries a wave takes by the graph's size, and edges found, failed and quick-rejected side by side."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle import kernelize_csr  # noqa: E402
from paper_2212_00574_amd import inputs  # noqa: E402
from paper_2212_00574_amd.binding import Kernelizer  # noqa: E402

from test_gpu_parity import check_same, run_csr  # noqa: E402

# class sizes, p, vertices joined to every other class (long rows)
CASES = {
    "long rows": ([3, 600, 500, 40], 0.02, 3),
    "rows at the table's limit": ([256, 257, 256, 20], 0.5, 2),
    "three classes": ([40, 50, 60], 0.2, 0),
    "two classes": ([40, 50], 0.2, 0),
    "cascade": ([60, 70, 64, 80, 75, 66], 0.15, 0),
    "64 classes": ([7] * 64, 0.5, 0),
    "70 classes": ([8] * 70, 0.55, 1),
    "300 classes": ([3] * 300, 0.75, 0),
    "32 entries a wave": ([150] * 6, 0.45, 0),
    "64 entries a wave": ([215] * 6, 0.45, 0),
}


@pytest.mark.parametrize("name", list(CASES))
def test_csr_edge(name):
    sizes, p, hubs = CASES[name]
    kz = Kernelizer(0)
    for seed in (0, 1):
        adj, colour = inputs.make_graph(sizes, p, seed=seed, gid=3, plant=seed == 1).dense()
        for h in range(hubs):
            adj[h, colour != colour[h]] = adj[colour != colour[h], h] = 1
        rp, ci = inputs.dense_to_csr(adj)
        res, vm, em = run_csr(kz, rp, ci, colour, len(sizes), "%s/%d" % (name, seed))
        check_same(res, kernelize_csr(rp, ci, colour, len(sizes)), vm, em, name)
    kz.close()
