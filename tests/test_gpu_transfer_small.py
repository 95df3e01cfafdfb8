"""Prolongation on small aggregates, which fewer workgroups share: one to four of them per aggregate half."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import Case, announce, need_gpu
from paper_1601_03184_amd import inputs, mrhs
from test_gpu_transfer import coarse_to_native, per_rhs_rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,agg", [([3, 2, 2, 2], [1, 1, 1, 1]), ([4, 4, 2, 4], [2, 2, 2, 2]), ([4, 4, 2, 3], [4, 2, 1, 3]),
                                   ([4, 4, 4, 2], [4, 2, 2, 2]), ([4, 3, 4, 2], [4, 3, 2, 2])])
@pytest.mark.parametrize("n_tv,n,S", [(5, 3, 4), (6, 17, 8), (1, 1, 1)])
def test_prolong_small_aggregates(L, agg, n_tv, n, S):
    need_gpu()
    announce("prolong small L=%s agg=%s n_tv=%d n=%d S=%d" % (L, agg, n_tv, n, S))
    op = Case(L, 0.3, 471, -0.2).op([1, 1, 1, 1], agg=agg, prec=mrhs.PREC_F32, short_len=S)
    qn = op.pack(torch.from_numpy(inputs.test_vectors(L, n_tv, 472) / np.sqrt(12.0 * np.prod(agg))))
    qin = op.unpack(qn, n_tv).cpu().numpy()
    rng = np.random.default_rng(473)
    z = (rng.standard_normal((n, op.n_agg, 2, n_tv)) + 1j * rng.standard_normal((n, op.n_agg, 2, n_tv))).astype(np.complex64)
    out = op.empty(n)
    out.fill_(float("nan"))
    mrhs.prolong_mrhs(op.handle, qn, mrhs.DTYPE_F32, n_tv, coarse_to_native(z.astype(np.complex128), (n + 3) // 4 * 4), out,
                      mrhs.DTYPE_F32, n)
    # FP32 products and sums over at most 6 vectors
    assert per_rhs_rel(op.unpack(out, n).cpu().numpy(), oracle.prolong(L, agg, qin, z.astype(np.complex128))) < 1e-5
    assert np.all(op.unpack(out, (n + S - 1) // S * S).cpu().numpy()[n:] == 0)
    op.close()
