"""Dominance over the row layouts its kernels are chosen by (rows in LDS or memory, 16, 32 or 64 lanes a row, one or
several words a lane) and over sparse and dense graphs, whose tests differ, against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle import dom_edge, dom_vertex  # noqa: E402
from paper_2212_00574_amd import inputs  # noqa: E402
from paper_2212_00574_amd.binding import KZ_DOM_EDGE, KZ_DOM_VERTEX, Kernelizer  # noqa: E402


@pytest.mark.parametrize("n,R", [(130, 4), (130, 5), (130, 8), (130, 9), (130, 16), (130, 17), (130, 32), (700, 32), (130, 33), (130, 64), (130, 65), (130, 256),
                                 (130, 257), (130, 1024), (1102, 18), (1103, 18)])
def test_row_layouts(n, R):
    kz = Kernelizer(0)
    rng = np.random.default_rng(n + R)
    for p in ((0.02, 0.3, 0.97) if n < 1000 else (0.995,)):
        print("dominance rows", n, R, p, flush=True)
        adj = np.triu((rng.random((n, n)) < p).astype(np.uint8), 1)
        adj |= adj.T
        rows = np.zeros((n, R), np.uint64)
        packed = inputs.dense_to_rows(adj)
        rows[:, :packed.shape[1]] = packed
        t = torch.from_numpy(rows.view(np.int64)).cuda()
        want, alive, ref = dom_vertex(adj)
        vm, em, res = kz.dominance(t, KZ_DOM_VERTEX)
        torch.cuda.synchronize()
        assert np.array_equal(vm.cpu().numpy(), alive), (n, R, p)
        assert np.array_equal(inputs.rows_to_dense(em.cpu().numpy()[:, :packed.shape[1]], n), want), (n, R, p)
        assert (res["sweeps"], res["events"], res["deleted_edges"]) == (ref["sweeps"], ref["steps"], ref["deleted_edges"])
        want, ref = dom_edge(adj)
        vm, em, res = kz.dominance(t, KZ_DOM_EDGE)
        torch.cuda.synchronize()
        assert np.array_equal(inputs.rows_to_dense(em.cpu().numpy()[:, :packed.shape[1]], n), want), (n, R, p)
        assert (res["sweeps"], res["deleted_edges"]) == (ref["sweeps"], ref["deleted_edges"]), (n, R, p)
    kz.close()
