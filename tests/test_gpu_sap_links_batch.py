"""A batch whose links are staged in LDS for every instance: blocks smaller than the batch's largest, with
link boxes and idle lanes of their own."""
import pytest
import torch

import oracle
from gpu_helpers import Case, announce, need_gpu, per_rhs_rel
from paper_1601_03184_amd import inputs, mrhs

pytestmark = pytest.mark.gpu

F64, F32, F16 = mrhs.PREC_F64, mrhs.PREC_F32, mrhs.PREC_F32_F16STORE
TOL = {F64: 1e-12, F32: 1e-5, F16: 5e-3}
# the largest block (256 sites) has the largest boxes: 192 + 256 + 256 + 192 links in the four directions, of
# which the first one, two and four fit at tiles 1, 2 and 4
SHAPES = [([8, 4, 4, 8], [4, 4, 4, 4]), ([6, 6, 6, 6], [3, 3, 3, 3]), ([4, 4, 4, 4], [1, 2, 4, 2]), ([4, 4, 2, 4], [2, 2, 2, 4])]


@pytest.mark.parametrize("prec,tile", [(F64, 1), (F64, 2), (F32, 1), (F32, 2), (F32, 4), (F16, 1), (F16, 4)])
def test_staged_links_of_uneven_blocks(prec, tile):
    need_gpu()
    announce("sap staged links batch prec=%d tile=%d" % (prec, tile))
    n, cases, ops, bs, xs = 6, [], [], [], []
    for L, block in SHAPES:
        case = Case(L, 0.3, 361, -0.1)
        op = case.op(block, prec=prec, short_len=4)
        mrhs.mrhs_set_tiles(op.handle, tile, 0)
        cases.append(case)
        ops.append(op)
        bs.append(op.pack(torch.from_numpy(inputs.test_vectors(L, n, 362))))
        xs.append(op.empty(n))
    hs = [op.handle for op in ops]
    need = mrhs.mrhs_batched_workspace_bytes(hs, [n] * len(ops))
    ws = torch.full((need + 4096,), 171, dtype=torch.uint8, device="cuda")
    mrhs.sap_smooth_mrhs_batched(hs, bs, xs, [n] * len(ops), 2, 3, ws[:need])
    assert torch.all(ws[need:] == 171)
    for (L, block), case, op, b, x in zip(SHAPES, cases, ops, bs, xs):
        ref = oracle.sap(L, block, case.U, case.A, op.unpack(b, n).cpu().numpy(), 2, 3)
        assert per_rhs_rel(op.unpack(x, n).cpu().numpy(), ref) < TOL[prec]
        op.close()
