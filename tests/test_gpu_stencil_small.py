"""The stencil on blocks of up to eight sites, where a workgroup takes two groups of right-hand sides, and of
a few more: every number of groups, ragged ones among them."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import Case, announce, need_gpu, per_rhs_rel
from paper_1601_03184_amd import inputs, mrhs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol", [(mrhs.PREC_F32, 1e-5), (mrhs.PREC_F32_F16STORE, 1e-3)])
@pytest.mark.parametrize("L,block", [([3, 2, 4, 2], [1, 1, 1, 1]), ([4, 3, 2, 2], [1, 3, 1, 1]), ([4, 4, 2, 4], [2, 2, 1, 2]),
                                     ([6, 3, 2, 2], [3, 3, 1, 1]), ([4, 4, 4, 2], [2, 2, 2, 2])])
@pytest.mark.parametrize("n", [1, 4, 5, 8, 11, 12])
def test_stencil_small_blocks(L, block, n, prec, tol):
    need_gpu()
    announce("stencil small L=%s block=%s n=%d prec=%d" % (L, block, n, prec))
    case = Case(L, 0.3, 461, -0.1)
    op = case.op(block, prec=prec, short_len=4)
    x = op.pack(torch.from_numpy(inputs.test_vectors(L, n, 462)))
    xin = op.unpack(x, n).cpu().numpy()
    y = torch.full((x.numel() + 64,), float("nan"), dtype=x.dtype, device="cuda")
    mrhs.dirac_apply_mrhs(op.handle, x, y[:x.numel()], n)
    # FP32 sums of about 100 terms; one rounding to binary16 (2^-11 relative at most)
    assert per_rhs_rel(op.unpack(y[:x.numel()], n).cpu().numpy(), oracle.dirac(L, case.U, case.A, xin)) < tol
    assert np.all(op.unpack(y[:x.numel()], (n + 3) // 4 * 4).cpu().numpy()[n:] == 0)
    assert torch.all(torch.isnan(y[x.numel():]))
    op.close()
