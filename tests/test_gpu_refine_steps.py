"""A refinement pass equals its separate calls, bit for bit: where the smoother's last sweep writes
over the test vectors and where its result is copied (no or one sweep, odd block counts)."""
import numpy as np
import pytest
import torch

from gpu_helpers import Case, announce, need_gpu
from paper_1601_03184_amd import inputs, mrhs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_sap", [0, 1, 2, 3])
@pytest.mark.parametrize("L,block,prec,n,solver", [
    ([8, 4, 4, 8], [4, 4, 4, 4], mrhs.PREC_F32, 7, 0),
    ([8, 4, 4, 8], [4, 4, 4, 4], mrhs.PREC_F32_F16STORE, 5, 1),
    ([6, 2, 2, 4], [2, 2, 2, 2], mrhs.PREC_F64, 4, 0),     # three blocks in a direction
])
def test_refine_is_its_steps(L, block, prec, n, solver, n_sap):
    need_gpu()
    announce("refine steps L=%s prec=%d n=%d solver=%d n_sap=%d" % (L, prec, n, solver, n_sap))
    op = Case(L, 0.3, 391, -0.2).op(block, prec=prec, short_len=4)
    if solver:
        mrhs.mrhs_set_block_solver(op.handle, mrhs.BLOCK_EO_MR)
    q = inputs.test_vectors(L, n, 392) / np.sqrt(12.0 * np.prod(block))
    Q = op.pack(torch.from_numpy(q), mrhs.DTYPE_F32)
    Dc = torch.zeros(op.n_agg * 9 * (2 * n) ** 2 * 2, dtype=torch.float32, device="cuda")
    mrhs.coarse_op_build(op.handle, Q, mrhs.DTYPE_F32, n, Dc, None)
    V = op.pack(torch.from_numpy(inputs.test_vectors(L, n, 393)))
    b = V.clone()
    ws = torch.empty(mrhs.mrhs_refine_workspace_bytes(op.handle, n, 4), dtype=torch.uint8, device="cuda")
    mrhs.setup_refine_mrhs(op.handle, V, n, Q, mrhs.DTYPE_F32, Dc, n_sap, 3, 4, 0.05, ws)
    vc, uc, x = op.coarse_empty(n, n), op.coarse_empty(n, n), op.empty(n)
    gm = torch.empty(mrhs.mrhs_coarse_solve_workspace_bytes(op.handle, n, n, 4), dtype=torch.uint8, device="cuda")
    mrhs.restrict_mrhs(op.handle, Q, mrhs.DTYPE_F32, n, b, op.dtype, vc, n)
    mrhs.coarse_solve_mrhs(op.handle, Dc, n, vc, uc, n, 4, 0.05, gm)
    mrhs.prolong_mrhs(op.handle, Q, mrhs.DTYPE_F32, n, uc, x, op.dtype, n)
    mrhs.sap_smooth_mrhs_guess(op.handle, b, x, n, n_sap, 3, op.workspace(n))
    assert torch.equal(V, x)
    op.close()
