"""A served request whose rows are malformed gets its status in every job of a
slot, not in the slot's first alone: one slot, valid requests and ones with an
asymmetric pair, a self-loop, an edge inside a class and a padding bit in turn,
passes run by one workgroup and shared."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle import kernelize_bitset  # noqa: E402
from paper_2212_00574_amd import inputs  # noqa: E402
from paper_2212_00574_amd.binding import (Kernelizer, Server, kz_batch_get_config,  # noqa: E402
                                          kz_batch_set_config)

SIZES = [70, 40, 30]  # rows of 4 words: class 0's in 0 and 1, class 1's in 2, class 2's in 3


def word(a, b):
    start, first = [0, 70, 110], [0, 2, 3]
    c = max(i for i in range(3) if start[i] <= b)
    return a, first[c] + (b - start[c]) // 64, np.uint64(1 << (b - start[c]) % 64)


def flip(rows, a, b):
    u, w, bit = word(a, b)
    rows[u, w] ^= bit


def spoil(rows, what):
    if what == "asymmetric":
        flip(rows, 5, 80)
    elif what == "loop":
        flip(rows, 9, 9)
    elif what == "inside":
        flip(rows, 3, 4)
        flip(rows, 4, 3)
    elif what == "padding":
        rows[7, 2] ^= np.uint64(1) << np.uint64(45)


@pytest.mark.parametrize("share", [0, 1])
def test_row_errors_in_a_reused_slot(share):
    kz = Kernelizer(0)
    try:
        kz_batch_set_config(kz.ctx, dict(kz_batch_get_config(kz.ctx), share=share))
        srv = Server(kz, arena_bytes=16 << 20, max_slots=1)
        for i, what in enumerate(["", "asymmetric", "loop", "", "inside", "padding", ""]):
            rows, colour, lay = inputs.make_graph(SIZES, 0.6, seed=61, gid=i, shuffle=False).bitset()
            assert lay.R == 4
            rows = rows.copy()
            spoil(rows, what)
            want = kernelize_bitset(rows, colour, 3)["status"]
            assert want == {"": 0, "asymmetric": -4, "loop": -5, "inside": -3, "padding": -1}[what]
            r = torch.from_numpy(rows.view(np.int64)).cuda()
            c = torch.from_numpy(colour).cuda()
            vm = torch.empty(lay.n, dtype=torch.uint8, device="cuda")
            em = torch.empty_like(r)
            ticket = srv.submit(r, c, 3, vm, em)
            assert ticket is not None
            t0 = time.time()
            res = None
            while res is None and time.time() - t0 < 60:
                res = srv.poll(ticket)
            assert res is not None and res["status"] == want, (i, what, res)
        srv.close()
    finally:
        kz.close()
