"""A session launch with nothing left ends for the single-graph lane's slices
that share its hardware queue: with an idle time and a lease of a second,
rounds of small and large requests end long before either, with the oracle's
masks, and the small requests after such an end start a launch of their own."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle import kernelize_bitset  # noqa: E402
from paper_2212_00574_amd import inputs  # noqa: E402
from paper_2212_00574_amd.binding import Kernelizer, Server  # noqa: E402

DEV = torch.device("cuda", 0)


@pytest.mark.parametrize("workers", [1, 8])
def test_idle_session_ends_for_the_other_lane(workers):
    kz = Kernelizer(0)
    srv = Server(kz, 256 << 20, max_slots=64, stream=torch.cuda.Stream())
    try:
        srv.configure(split_n=300, idle_us=1000000, lease_us=1000000, workers=workers)
        graphs = []
        for i in range(24):
            sizes = [40] * 5 if i % 3 else [90] * 6
            g = inputs.make_graph(sizes, 0.2 + 0.02 * i, seed=77, gid=i, plant=False, shuffle=False)
            rows, colour, lay = g.bitset()
            graphs.append((rows, colour, len(sizes), lay, kernelize_bitset(rows, colour, len(sizes))))
        for turn in range(4):
            reqs = []
            for rows, colour, k, lay, _ in graphs:
                reqs.append((torch.from_numpy(rows.view(np.int64).reshape(-1).copy()).to(DEV),
                             torch.from_numpy(colour).to(DEV), k,
                             torch.full((lay.n,), 9, dtype=torch.uint8, device=DEV),
                             torch.full((lay.n * lay.R,), -1, dtype=torch.int64, device=DEV)))
            torch.cuda.synchronize()
            t0 = time.time()
            tickets = [srv.submit(*r) for r in reqs]
            res = [None] * len(reqs)
            while any(x is None for x in res):
                for j, t in enumerate(tickets):
                    if res[j] is None:
                        res[j] = srv.poll(t)
                assert time.time() - t0 < 30, "requests did not complete"
            spent = time.time() - t0
            print("workers", workers, "turn", turn, "%.1f ms" % (spent * 1e3), flush=True)
            for i, (r, x) in enumerate(zip(reqs, res)):
                rows, colour, k, lay, ref = graphs[i]
                assert x["status"] == 0 and x["rounds"] == ref["rounds"], (turn, i)
                assert np.array_equal(r[3].cpu().numpy(), ref["vmask"]), (turn, i)
                assert np.array_equal(r[4].cpu().numpy().view(np.uint64).reshape(lay.n, lay.R), ref["emask"]), (turn, i)
            assert spent < 0.5, "a request waited for the session launch"
    finally:
        srv.close()
        kz.close()
