"""The status of block Gram-Schmidt names the first aggregate half that is rank-deficient."""
import numpy as np
import pytest
import torch

from gpu_helpers import Case, announce, need_gpu
from paper_1601_03184_amd import inputs, mrhs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("halves", [[], [(5, 1)], [(0, 0)], [(15, 1)], [(9, 0), (6, 1)], [(13, 0), (2, 1), (2, 0)]])
@pytest.mark.parametrize("qdt", [mrhs.DTYPE_F64, mrhs.DTYPE_F32])
def test_status_is_the_first_half(halves, qdt):
    need_gpu()
    announce("gs status %s qdt=%d" % (halves, qdt))
    L, agg = [4, 4, 4, 4], [2, 2, 2, 2]                       # 16 aggregates, 32 halves
    op = Case(L, 0.3, 301, -0.2).op(agg, prec=mrhs.PREC_F64, short_len=4)
    v = inputs.test_vectors(L, 4, 303)
    c = inputs.site_coords(L)
    agg_of = (c // 2) @ np.array([1, 2, 4, 8])
    for i, h in halves:                                       # the last vector depends on two others there
        at = agg_of == i
        v[3][at, 2 * h:2 * h + 2] = 0.5 * v[0][at, 2 * h:2 * h + 2] - 2j * v[2][at, 2 * h:2 * h + 2]
    status = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    mrhs.block_orthonormalize(op.handle, op.pack(torch.from_numpy(v)), mrhs.DTYPE_F64, op.empty(4, qdt), qdt, 4, status,
                              op.workspace(4))
    assert int(status.item()) == min([1 + 2 * i + h for i, h in halves], default=0)
    op.close()
