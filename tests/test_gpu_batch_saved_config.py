"""A saved configuration of 4 or 8 waves costs no time over one of 16: the waves
are kept for such configurations and a workgroup has 16 whatever they say.  (Run
with 4 waves, the batch below took eight times as long.)"""
import time

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2212_00574_amd import inputs  # noqa: E402
from paper_2212_00574_amd.binding import (Batch, BatchKernelizer, Kernelizer, kz_batch_get_config,  # noqa: E402
                                          kz_batch_set_config)


def test_saved_waves_cost_no_time():
    kz = Kernelizer(0)
    try:
        graphs = [inputs.make_graph([96] * 12, 0.22, seed=71, gid=i, shuffle=False) for i in range(48)]
        items = []
        for g in graphs:
            rows, colour, _ = g.bitset()
            items.append((rows, colour, 12))
        b = Batch(items, torch.device("cuda", 0))
        bk = BatchKernelizer(kz)
        took, masks = {}, {}
        for waves in (16, 4, 8):
            kz_batch_set_config(kz.ctx, dict(waves=waves, chunk=4, lpt=1, workgroups=0, share=0))
            assert kz_batch_get_config(kz.ctx)["waves"] == waves
            times = []
            for _ in range(6):
                t0 = time.perf_counter()
                bk.run(b)
                torch.cuda.synchronize()
                times.append(time.perf_counter() - t0)
            took[waves], masks[waves] = min(times[1:]), b.emask.clone()
        assert torch.equal(masks[16], masks[4]) and torch.equal(masks[16], masks[8])
        assert took[4] < 2 * took[16] and took[8] < 2 * took[16], took
    finally:
        kz.close()
