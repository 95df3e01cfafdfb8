"""The SAP's workspace needs the alignment of the arithmetic type and no more."""
import pytest
import torch

from gpu_helpers import Case, announce, need_gpu
from paper_1601_03184_amd import inputs, mrhs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,step", [(mrhs.PREC_F64, 8), (mrhs.PREC_F32, 4), (mrhs.PREC_F32_F16STORE, 4)])
@pytest.mark.parametrize("L,solver", [([8, 4, 4, 8], 0), ([12, 4, 4, 4], 0), ([8, 4, 4, 8], 1)])
def test_workspace_at_any_element(L, solver, prec, step):
    need_gpu()
    announce("sap workspace L=%s prec=%d solver=%d" % (L, prec, solver))
    op, n = Case(L, 0.3, 431, -0.1).op([4, 4, 4, 4], prec=prec, short_len=4), 5
    if solver:
        mrhs.mrhs_set_block_solver(op.handle, mrhs.BLOCK_EO_MR)
    b = op.pack(torch.from_numpy(inputs.test_vectors(L, n, 432)))
    need = mrhs.mrhs_workspace_bytes(op.handle, n)
    ws = torch.empty(need + 64, dtype=torch.uint8, device="cuda")
    assert ws.data_ptr() % 16 == 0
    xs = []
    for at in (0, step, 12 // step * step):
        x = op.empty(n)
        mrhs.sap_smooth_mrhs(op.handle, b, x, n, 3, 2, ws[at:at + need])
        xs.append(x)
    assert torch.equal(xs[0], xs[1]) and torch.equal(xs[0], xs[2])
    op.close()
