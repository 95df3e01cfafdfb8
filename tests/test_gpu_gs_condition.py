"""Block Gram-Schmidt on both sides of the condition limit below which one Cholesky pass is
taken (Q stored in FP32 or binary16): nearly parallel test vectors of growing condition."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import Case, announce, need_gpu, per_agg_half_rel
from paper_1601_03184_amd import inputs, mrhs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("qdt,tol", [(mrhs.DTYPE_F32, 1e-6), (mrhs.DTYPE_F16, 1e-3)])
@pytest.mark.parametrize("eps", [1.0, 0.1, 0.02, 1e-3])
@pytest.mark.parametrize("L,agg,n", [([8, 4, 4, 4], [4, 4, 4, 4], 32), ([4, 4, 4, 4], [2, 4, 2, 2], 17),
                                     ([6, 3, 3, 3], [3, 3, 3, 3], 16), ([4, 4, 4, 4], [2, 2, 2, 2], 1)])
def test_gs_condition(L, agg, n, eps, qdt, tol):
    need_gpu()
    announce("gs condition L=%s agg=%s n=%d eps=%g qdt=%d" % (L, agg, n, eps, qdt))
    op = Case(L, 0.3, 341, -0.2).op(agg, agg=agg, prec=mrhs.PREC_F32, short_len=4)
    # every vector a common one plus eps times its own: column-scaled condition number ~ sqrt(n) / eps,
    # so its square times n crosses 2^16 between eps = 0.1 and 0.02 at 32 vectors
    v = inputs.test_vectors(L, n + 1, 342)
    v = v[:1] + eps * v[1:]
    vn = op.pack(torch.from_numpy(v), mrhs.DTYPE_F64)
    status = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    Q = op.empty(n, qdt)
    mrhs.block_orthonormalize(op.handle, vn, mrhs.DTYPE_F64, Q, qdt, n, status, op.workspace(n))
    assert int(status.item()) == 0
    got = op.unpack(Q, n, qdt).cpu().numpy()
    # one rounding of each entry to the storage type (2^-25, 2^-12 relative), everything else in FP64
    assert per_agg_half_rel(got, oracle.block_gs(L, agg, v), L, agg) < tol
    op.close()
