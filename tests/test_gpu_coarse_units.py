"""The coarse operator at the edges of its work units: vector counts around the groups of four,
every short length, aggregates whose sites and faces do not fill a chunk of eight sites."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import Case, announce, need_gpu
from paper_1601_03184_amd import inputs, mrhs

pytestmark = pytest.mark.gpu

F64, F32 = mrhs.PREC_F64, mrhs.PREC_F32
D64, D32, D16 = mrhs.DTYPE_F64, mrhs.DTYPE_F32, mrhs.DTYPE_F16

CASES = [
    # (L, block, agg, prec, S, n, qdt)
    ([6, 3, 3, 6], [3, 3, 3, 3], [3, 3, 3, 3], F32, 4, 32, D32),   # 81 sites, faces of 27
    ([6, 3, 3, 3], [3, 3, 3, 3], [3, 3, 3, 3], F64, 4, 5, D64),
    ([4, 4, 2, 2], [2, 2, 2, 2], [2, 2, 2, 1], F32, 1, 3, D32),    # 8 sites: one chunk, faces of 4 and 8
    ([4, 2, 4, 2], [2, 2, 2, 2], [2, 1, 1, 2], F32, 2, 1, D32),    # 4 sites, one vector
    ([4, 4, 4, 4], [4, 4, 4, 4], [2, 4, 4, 2], F32, 8, 29, D16),
    ([8, 4, 4, 4], [4, 4, 4, 4], [4, 4, 4, 4], F32, 4, 4, D64),
    ([4, 4, 4, 4], [2, 2, 2, 2], [4, 4, 4, 4], F64, 4, 31, D32),   # one aggregate, its own neighbour
]


@pytest.mark.parametrize("L,block,agg,prec,S,n,qdt", CASES)
def test_coarse_units(L, block, agg, prec, S, n, qdt):
    need_gpu()
    announce("coarse units L=%s agg=%s n=%d S=%d" % (L, agg, n, S))
    case = Case(L, 0.3, 361, -0.2)
    op = case.op(block, agg=agg, prec=prec, short_len=S)
    qn = op.pack(torch.from_numpy(inputs.test_vectors(L, n, 362) / np.sqrt(12.0 * np.prod(agg))), qdt)
    qin = op.unpack(qn, n, qdt).cpu().numpy()
    size = op.n_agg * 9 * (2 * n) ** 2 * 2
    Dc = torch.full((size + 64,), float("nan"), dtype=torch.float32, device="cuda")
    mrhs.coarse_op_build(op.handle, qn, qdt, n, Dc[:size], None)
    got = Dc[:size].cpu().double().numpy().view(np.complex128).reshape(op.n_agg, 9, 2 * n, 2 * n)
    ref = oracle.coarse_op(L, agg, case.U, case.A, qin)
    for d in range(9):
        # FP32 products over 12 Va <= 3072 rows, D_c of order one
        assert np.linalg.norm(got[:, d] - ref[:, d]) < 1e-5 * np.linalg.norm(ref[:, d]), d
    assert torch.all(torch.isnan(Dc[size:]))
    op.close()
