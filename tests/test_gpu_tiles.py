"""The batched path's tile test (matrix products, pairs one per lane, miss counts) and its vertex test against the
oracle, bit for bit, at the sizes where they split: half and whole blocks, one, two and many words a class, more
words than a window, classes that end early, empty classes, and clique sizes far below the colour classes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle import fixpoint_rows  # noqa: E402
from paper_2212_00574_amd import inputs  # noqa: E402
from paper_2212_00574_amd.binding import Batch, BatchKernelizer, Kernelizer, kz_batch_set_config  # noqa: E402

DEV = torch.device("cuda", 0)

# class sizes, p, cliques below the class count (0: equal to it)
CASES = {
    "half blocks": ([20, 33, 64, 65, 97, 32, 1], 0.5, (0, 1, 3)),
    "three words": ([129, 150, 192, 191, 130], 0.25, (0, 1)),
    "a window": ([448, 447, 300, 200], 0.12, (0, 1)),
    "past a window": ([449, 512, 500, 513], 0.1, (0, 1)),
    "ends early": ([700, 640, 690, 650], 0.5, (0, 1)),
    "sparse": ([400, 390, 380, 200], 0.06, (0, 1)),
    "empty class": ([60, 0, 90, 70, 65], 0.6, (0, 1, 2)),
    "many classes": ([6] * 64, 0.85, (0, 8, 40, 61)),
    "cascade": ([60, 70, 64, 80, 75, 66], 0.17, (0, 1)),
    "two classes": ([100, 40], 0.3, (0, 1)),
}


@pytest.mark.parametrize("waves", [4, 8, 16])
def test_tiles(waves):
    kz = Kernelizer(0)
    kz_batch_set_config(kz.ctx, dict(waves=waves, chunk=4, lpt=1, workgroups=0, share=0))
    graphs, names = [], []
    for name, (sizes, p, below) in CASES.items():
        for b in below:
            for seed in (0, 1):
                rows, colour, _ = inputs.make_graph(sizes, p, seed=seed, gid=len(names), plant=0 not in sizes and seed == 1,
                                                    shuffle=False).bitset()
                k = len(sizes)
                graphs.append((rows, colour, k, k - b if b else 0))
                names.append("%s/%d/%d" % (name, b, seed))
    print("tiles: waves", waves, len(graphs), "graphs", flush=True)
    batch = Batch(graphs, DEV)
    BatchKernelizer(kz).run(batch)
    torch.cuda.synchronize()
    res = batch.read_results()
    for i, (rows, colour, k, clique) in enumerate(graphs):
        ref, r = fixpoint_rows(rows, colour, k, clique=clique or k), res[i]
        got = [int(r[x]) for x in ("status", "rounds", "surviving_vertices", "surviving_edges", "edge_tests")]
        want = [ref[x] for x in ("status", "rounds", "surv_vertices", "surv_edges", "edge_tests")]
        assert got == want, (names[i], got, want)
        vm, em = batch.masks(i)
        assert np.array_equal(vm, ref["vmask"]) and np.array_equal(em, ref["emask"]), names[i]
    kz.close()
