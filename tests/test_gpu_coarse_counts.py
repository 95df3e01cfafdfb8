"""The coarse solve at the right-hand-side counts where its projection changes how many chunks a workgroup
takes: the oracle's solution, and a vector's result to the last bit whatever else is in the call."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import Case, announce, need_gpu
from paper_1601_03184_amd import mrhs
from test_gpu_transfer import coarse_from_native, coarse_to_native, per_rhs_rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 8, 10])          # the fused projection takes up to 8 basis vectors
@pytest.mark.parametrize("L,n_tv", [([8, 4, 4, 4], 3), ([8, 8, 4, 8], 20)])
def test_solve_counts(L, n_tv, m):
    need_gpu()
    announce("coarse counts L=%s n_tv=%d m=%d" % (L, n_tv, m))
    agg, ns = [4, 4, 4, 4], [1, 4, 5, 12, 16, 17, 32]
    op = Case(L, 0.3, 451, -0.2).op(agg, prec=mrhs.PREC_F32, short_len=4)
    rng, N2 = np.random.default_rng(452), 2 * n_tv
    cplx = lambda *s: (rng.standard_normal(s) + 1j * rng.standard_normal(s)).astype(np.complex64)
    D = 0.5 / N2 ** 0.5 * cplx(op.n_agg, 9, N2, N2)
    D[:, 0, range(N2), range(N2)] += 4.0
    b = cplx(max(ns), op.n_agg, 2, n_tv)
    Dc = torch.from_numpy(D.astype(np.complex64).view(np.float32)).cuda()
    ref = oracle.coarse_gmres(L, agg, D.astype(np.complex128), b[:1].astype(np.complex128), m)
    ref = ref[0] if isinstance(ref, tuple) else ref
    first = []
    for n in ns:
        bc = coarse_to_native(b[:n], (n + 3) // 4 * 4)
        uc = torch.full_like(bc, float("nan"))
        ws = torch.empty(mrhs.mrhs_coarse_solve_workspace_bytes(op.handle, n_tv, n, m), dtype=torch.uint8, device="cuda")
        mrhs.coarse_solve_mrhs(op.handle, Dc, n_tv, bc, uc, n, m, 0.0, ws)
        u = coarse_from_native(uc, op.n_agg, n_tv, n)
        first.append(u[0])
        # FP32 vectors and products: rounding of the operator's 9 N2 <= 360 terms, condition below 10
        assert per_rhs_rel(u[:1], ref.reshape(u[:1].shape)) < 1e-4
    for u in first[1:]:
        assert np.array_equal(u, first[0])
    op.close()
