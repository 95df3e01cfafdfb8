"""Restriction and prolongation at the edges of their tiles: one and two 16-wide tiles of test
vectors and of right-hand sides, aggregates whose sites do not fill the last 16-row block."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import Case, announce, need_gpu
from paper_1601_03184_amd import inputs, mrhs
from test_gpu_transfer import coarse_from_native, coarse_to_native, per_rhs_rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,agg", [([6, 3, 6, 3], [3, 3, 3, 3]), ([4, 2, 2, 4], [2, 1, 2, 2]), ([4, 4, 4, 4], [4, 4, 4, 4])])
@pytest.mark.parametrize("n_tv,n", [(16, 16), (17, 16), (16, 17), (17, 17), (1, 1), (31, 5)])
def test_restrict_prolong_tile_edges(L, agg, n_tv, n):
    need_gpu()
    announce("restrict/prolong tiles L=%s agg=%s n_tv=%d n=%d" % (L, agg, n_tv, n))
    op = Case(L, 0.3, 331, -0.2).op(agg, agg=agg, prec=mrhs.PREC_F32, short_len=4)
    q = inputs.test_vectors(L, n_tv, 332) / np.sqrt(12.0 * np.prod(agg))
    qn = op.pack(torch.from_numpy(q))
    qin = op.unpack(qn, n_tv).cpu().numpy()
    yn = op.pack(torch.from_numpy(inputs.test_vectors(L, n, 333)))
    yin = op.unpack(yn, n).cpu().numpy()
    yc = op.coarse_empty(n_tv, n)
    yc.fill_(float("nan"))
    mrhs.restrict_mrhs(op.handle, qn, mrhs.DTYPE_F32, n_tv, yn, mrhs.DTYPE_F32, yc, n)
    got = coarse_from_native(yc, op.n_agg, n_tv, n)
    # FP32 products and sums over 6 Va <= 1536 rows: rounding well below 1e-5 of the result
    assert per_rhs_rel(got, oracle.restrict(L, agg, qin, yin)) < 1e-5
    rng = np.random.default_rng(334)
    z = rng.standard_normal((n, op.n_agg, 2, n_tv)) + 1j * rng.standard_normal((n, op.n_agg, 2, n_tv))
    z = z.real.astype(np.float32) + 1j * z.imag.astype(np.float32)
    out = op.empty(n)
    out.fill_(float("nan"))
    mrhs.prolong_mrhs(op.handle, qn, mrhs.DTYPE_F32, n_tv, coarse_to_native(z, (n + 3) // 4 * 4), out, mrhs.DTYPE_F32, n)
    assert per_rhs_rel(op.unpack(out, n).cpu().numpy(), oracle.prolong(L, agg, qin, z.astype(np.complex128))) < 1e-5
    full = op.unpack(out, (n + 3) // 4 * 4).cpu().numpy()
    assert np.all(full[n:] == 0)
    op.close()
