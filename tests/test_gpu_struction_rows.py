"""G' against the oracle where its rows' kernel splits: |A| and the C nodes
around multiples of 64 (the transposed words of the A rows, the blocks of the C
rows), blocks over several words, an output wider and longer than G', and one
that does not hold it (refused, nothing written past what the caller gave)."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle import struction  # noqa: E402
from paper_2212_00574_amd import binding, inputs  # noqa: E402

DEV = "cuda:0"


def graph(n, na, p, seed):
    """Random graph whose vertex 0 has degree na."""
    rng = np.random.default_rng(seed)
    a = np.triu((rng.random((n, n)) < p).astype(np.uint8), 1)
    a[0] = 0
    a[0, 1 + rng.permutation(n - 1)[:na]] = 1
    return a + a.T


@pytest.mark.parametrize("n,na,p", [(70, 0, 0.3), (130, 1, 0.9), (130, 63, 0.5), (130, 64, 0.5), (130, 65, 0.5),
                                    (200, 128, 0.95), (200, 199, 0.5), (257, 30, 0.9)])
@pytest.mark.parametrize("room", [0, 1, 77])
def test_outputs_at_word_edges(n, na, p, room):
    adj = graph(n, na, p, 7 * n + na)
    ref, rmap = struction(adj, 0)
    npr = ref.shape[0]
    R, RP, cap = (n + 63) // 64, (npr + 63) // 64 + room, npr + room
    rows = torch.from_numpy(inputs.dense_to_rows(adj).view(np.int64)).to(DEV)
    k = binding.Kernelizer(0)
    try:
        L, C = binding.LIB, binding.C
        size = C.c_size_t(0)
        assert L.kz_struction_workspace_bytes(n, R, C.byref(size)) == 0
        ws = torch.empty(size.value, dtype=torch.uint8, device=DEV)
        stream = torch.cuda.current_stream().cuda_stream

        def call(nodes, words):
            out = torch.full((max(cap, 1), max(RP, 1)), -1, dtype=torch.int64, device=DEV)
            mp = torch.full((max(cap, 1), 2), -7, dtype=torch.int32, device=DEV)
            res = binding.kz_struction_result()
            st = L.kz_struction(k.ctx, n, rows.data_ptr(), R, 0, ws.data_ptr(), size.value, out.data_ptr(), words,
                                nodes, mp.data_ptr(), stream, C.byref(res))
            torch.cuda.synchronize()
            assert (res.nodes, res.a_nodes, res.c_nodes) == (npr, na, npr - na)
            return st, out.cpu().numpy(), mp.cpu().numpy()

        st, out, mp = call(cap, RP)
        assert st == 0
        if npr:
            assert np.array_equal(mp[:npr], rmap)
            assert np.array_equal(inputs.rows_to_dense(out[:npr, :(npr + 63) // 64], npr), ref)
            assert not out[:npr, (npr + 63) // 64:].any()
        assert (out[npr:cap] == -1).all() and (mp[npr:cap] == -7).all()
        if room == 0 and npr:  # a node, then a word short
            for nodes, words in ((npr - 1, RP), (npr, RP - 1)):
                st, out, mp = call(nodes, words)
                assert st == -6 and (out == -1).all() and (mp == -7).all()
    finally:
        k.close()
