"""Block Gram-Schmidt does not depend on the scale of V, down to squared norms below the smallest normal
double."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import Case, announce, need_gpu, per_agg_half_rel
from paper_1601_03184_amd import inputs, mrhs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [1e-150, 1e-156, 3e-157])
@pytest.mark.parametrize("L,agg,n", [([4, 4, 4, 4], [2, 2, 2, 2], 8), ([4, 4, 4, 4], [4, 4, 4, 4], 20)])
def test_gs_small_vectors(L, agg, n, scale):
    need_gpu()
    announce("gs scale %g n=%d" % (scale, n))
    op = Case(L, 0.3, 301, -0.2).op(agg, prec=mrhs.PREC_F64, short_len=4)
    v = inputs.test_vectors(L, n, 305)
    status = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    Q = op.empty(n, mrhs.DTYPE_F64)
    mrhs.block_orthonormalize(op.handle, op.pack(torch.from_numpy(v * scale)), mrhs.DTYPE_F64, Q, mrhs.DTYPE_F64, n, status,
                              op.workspace(n))
    assert int(status.item()) == 0
    # squared norms of 1e-311 hold 40 bits (2^-1074 is 5e-324); the second pass works on columns of norm one
    got = op.unpack(Q, n, mrhs.DTYPE_F64).cpu().numpy()
    assert per_agg_half_rel(got, oracle.block_gs(L, agg, v), L, agg) < 1e-9
    op.close()
