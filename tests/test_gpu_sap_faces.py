"""The SAP's face buffers: block shapes down to one site thick, every short length and ragged
groups, both block solvers, from zero and from a guess; nothing is written outside the
workspace that the size query asks for."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import Case, announce, need_gpu, per_rhs_rel
from paper_1601_03184_amd import inputs, mrhs

pytestmark = pytest.mark.gpu

F64, F32, F16 = mrhs.PREC_F64, mrhs.PREC_F32, mrhs.PREC_F32_F16STORE
TOL = {F64: 1e-12, F32: 1e-5, F16: 5e-3}
GUARD = 4096

CASES = [
    # (L, block, prec, S, n, n_sap, n_mr, tile, solver)
    ([4, 4, 2, 2], [1, 2, 2, 2], F64, 4, 5, 2, 3, 2, 0),   # one site thick: on both faces
    ([2, 4, 4, 2], [1, 1, 2, 2], F32, 2, 3, 3, 2, 1, 0),
    ([2, 2, 2, 2], [1, 1, 1, 1], F32, 1, 2, 2, 2, 1, 0),   # one site per block: all faces at once
    ([8, 4, 4, 4], [4, 2, 2, 4], F32, 8, 9, 3, 2, 4, 0),   # two groups of eight; a direction of one block
    ([8, 4, 4, 8], [4, 4, 4, 4], F32, 4, 6, 3, 0, 4, 0),   # no MR step
    ([6, 6, 12, 12], [3, 3, 3, 3], F32, 4, 5, 2, 3, 4, 0),  # odd extents, even block counts
    ([4, 4, 4, 4], [2, 2, 2, 2], F16, 4, 7, 3, 2, 2, 1),   # even-odd
    ([8, 4, 8, 4], [4, 4, 4, 4], F32, 4, 6, 3, 0, 4, 1),
    ([4, 4, 8, 4], [2, 4, 4, 2], F64, 2, 3, 3, 2, 1, 1),
    # odd block counts: neighbours of the own colour, face buffers alternating from sweep to sweep
    ([6, 6, 2, 2], [2, 2, 2, 2], F32, 4, 5, 4, 2, 4, 0),
    ([6, 2, 10, 4], [2, 2, 2, 2], F64, 4, 3, 3, 2, 2, 0),
    ([3, 3, 4, 4], [1, 1, 2, 2], F64, 1, 2, 3, 2, 1, 0),   # three blocks, one site thick
    ([3, 5, 2, 2], [1, 1, 2, 1], F32, 2, 3, 3, 2, 2, 0),
    ([12, 4, 4, 8], [4, 4, 4, 4], F16, 4, 6, 3, 3, 4, 0),
    ([6, 4, 6, 2], [2, 2, 2, 2], F32, 4, 4, 4, 2, 2, 1),
    ([4, 6, 2, 10], [2, 2, 2, 2], F64, 2, 2, 3, 2, 1, 1),
]


@pytest.mark.parametrize("L,block,prec,S,n,n_sap,n_mr,tile,solver", CASES)
@pytest.mark.parametrize("guess", [False, True])
def test_sap_faces(L, block, prec, S, n, n_sap, n_mr, tile, solver, guess):
    need_gpu()
    announce("sap faces L=%s block=%s prec=%d S=%d n=%d solver=%d guess=%d" % (L, block, prec, S, n, solver, guess))
    case = Case(L, 0.3, 351, -0.1)
    op = case.op(block, prec=prec, short_len=S)
    mrhs.mrhs_set_tiles(op.handle, tile, 0)
    if solver:
        mrhs.mrhs_set_block_solver(op.handle, mrhs.BLOCK_EO_MR)
    v = inputs.test_vectors(L, n, 352)
    b = op.pack(torch.from_numpy(v))
    x = op.pack(torch.from_numpy(0.3 * inputs.test_vectors(L, n, 353)))
    bin_, x0 = op.unpack(b, n).cpu().numpy(), op.unpack(x, n).cpu().numpy()
    need = mrhs.mrhs_workspace_bytes(op.handle, n)
    ws = torch.full((need + GUARD,), 171, dtype=torch.uint8, device="cuda")
    call = mrhs.sap_smooth_mrhs_guess if guess else mrhs.sap_smooth_mrhs
    call(op.handle, b, x, n, n_sap, n_mr, ws[:need])
    ref = oracle.sap(L, block, case.U, case.A, bin_, n_sap, n_mr, x0=x0 if guess else None, eo=bool(solver))
    got = op.unpack(x, n).cpu().numpy()
    if np.linalg.norm(ref) == 0:
        assert np.all(got == 0)  # no MR step from zero
    else:
        assert per_rhs_rel(got, ref) < TOL[prec]
    assert torch.all(ws[need:] == 171)
    op.close()
