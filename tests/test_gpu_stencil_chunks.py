"""The stencil and the FP64 residual on blocks that are cut into chunks, fill one or leave lanes
idle: hops that stay in a chunk, leave it for another one, cross a block face or wrap around."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import Case, announce, need_gpu, per_rhs_rel
from paper_1601_03184_amd import inputs, mrhs

pytestmark = pytest.mark.gpu

F64, F32, F16 = mrhs.PREC_F64, mrhs.PREC_F32, mrhs.PREC_F32_F16STORE
TOL = {F64: 1e-12, F32: 1e-5, F16: 5e-3}

CASES = [
    # (L, block, prec, S, n)
    ([8, 4, 4, 8], [4, 4, 4, 4], F32, 4, 5),     # two chunks of 128 sites, eight of 32
    ([8, 2, 4, 6], [4, 2, 4, 6], F32, 4, 3),     # 192 sites: two chunks of 96
    ([6, 3, 3, 6], [3, 3, 3, 3], F16, 4, 9),     # 81 sites
    ([4, 4, 4, 4], [4, 4, 4, 4], F32, 4, 4),     # one block that wraps around in every direction
    ([4, 4, 2, 2], [1, 1, 1, 1], F32, 4, 7),     # one site per block
    ([5, 3, 7, 2], [5, 3, 7, 2], F32, 4, 6),     # 210 sites in odd extents
    ([8, 4, 4, 4], [4, 4, 4, 4], F64, 4, 4),
    ([8, 4, 4, 4], [4, 4, 4, 4], F16, 8, 11),
    ([4, 4, 4, 4], [2, 4, 4, 4], F32, 2, 3),
    ([4, 4, 4, 4], [4, 4, 4, 4], F64, 1, 2),
]


@pytest.mark.parametrize("L,block,prec,S,n", CASES)
def test_stencil_chunks(L, block, prec, S, n):
    need_gpu()
    announce("stencil chunks L=%s block=%s prec=%d S=%d n=%d" % (L, block, prec, S, n))
    case = Case(L, 0.3, 371, -0.1)
    op = case.op(block, prec=prec, short_len=S)
    x = op.pack(torch.from_numpy(inputs.test_vectors(L, n, 372)))
    b = op.pack(torch.from_numpy(inputs.test_vectors(L, n, 373)))
    xin, bin_ = op.unpack(x, n).cpu().numpy(), op.unpack(b, n).cpu().numpy()
    y = op.empty(n)
    y.fill_(float("nan"))
    mrhs.dirac_apply_mrhs(op.handle, x, y, n)
    assert per_rhs_rel(op.unpack(y, n).cpu().numpy(), oracle.dirac(L, case.U, case.A, xin)) < TOL[prec]
    full = op.unpack(y, (n + S - 1) // S * S).cpu().numpy()
    assert np.all(full[n:] == 0)
    out = torch.full((n,), float("nan"), dtype=torch.float64, device="cuda")
    mrhs.mrhs_residual_norms(op.handle, b, x, n, out, op.workspace(n))
    ref = oracle.residual_norms(L, case.U, case.A, bin_, xin)
    assert np.max(np.abs(out.cpu().numpy() - ref) / ref) < 1e-12
    op.close()


def test_residual_long_grid():
    """A grid of one workgroup per block (2048 blocks and more) against one per chunk (fewer
    right-hand sides), the same vectors."""
    need_gpu()
    L, block = [16, 16, 8, 8], [2, 2, 2, 2]
    announce("residual long grid L=%s" % L)
    case = Case(L, 0.3, 381, -0.1)
    op = case.op(block, prec=F32, short_len=4)
    n = 20
    x = op.pack(torch.from_numpy(inputs.test_vectors(L, n, 382)))
    b = op.pack(torch.from_numpy(inputs.test_vectors(L, n, 383)))
    many = torch.empty(n, dtype=torch.float64, device="cuda")
    mrhs.mrhs_residual_norms_noalloc(op.handle, b, x, n, many)
    few = torch.empty(4, dtype=torch.float64, device="cuda")
    mrhs.mrhs_residual_norms_noalloc(op.handle, b, x, 4, few)
    # FP64 sums in another order
    assert torch.max(torch.abs(many[:4] - few) / few) < 1e-13
    op.close()
