"""Two threads whose launches of one kernel take different amounts of LDS, on streams of their own."""
import threading

import pytest
import torch

from gpu_helpers import Case, announce, need_gpu
from paper_1601_03184_amd import inputs, mrhs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tile", [(mrhs.PREC_F64, 2), (mrhs.PREC_F32, 2), (mrhs.PREC_F32, 4)])
def test_two_block_sizes_at_once(prec, tile):
    need_gpu()
    announce("lds limit prec=%d tile=%d" % (prec, tile))
    work, n = [], 8
    # 256 and 192 sites per block: more than 64 KiB of LDS each, and not the same
    for L, block in (([8, 4, 4, 4], [4, 4, 4, 4]), ([8, 4, 4, 3], [4, 4, 4, 3])):
        op = Case(L, 0.3, 441, -0.1).op(block, prec=prec, short_len=4)
        mrhs.mrhs_set_tiles(op.handle, tile, 0)
        b = op.pack(torch.from_numpy(inputs.test_vectors(L, n, 442)))
        ref = op.empty(n)
        mrhs.sap_smooth_mrhs(op.handle, b, ref, n, 2, 2, op.workspace(n))
        work.append((op, b, ref))
    torch.cuda.synchronize()
    failed = []

    def run(op, b, ref):
        try:
            st, x, ws = torch.cuda.Stream(), op.empty(n), op.workspace(n)
            for _ in range(50):
                mrhs.sap_smooth_mrhs(op.handle, b, x, n, 2, 2, ws, stream=st)
            st.synchronize()
            if not torch.equal(x, ref):
                failed.append("results differ")
        except Exception as e:  # noqa: BLE001 - reported by the main thread
            failed.append(str(e))

    threads = [threading.Thread(target=run, args=w) for w in work]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed
    for op, _, _ in work:
        op.close()
