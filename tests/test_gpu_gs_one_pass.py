"""The rule that skips Gram-Schmidt's second Cholesky pass: at a condition where one pass alone would be
seen in the stored Q, and on both sides of the limit."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import Case, announce, need_gpu, per_agg_half_rel
from paper_1601_03184_amd import inputs, mrhs

pytestmark = pytest.mark.gpu


def limit_ratio(V, L, agg):
    """largest N sum_l |v_l|^2 sum_m |(R^-1)_lm|^2 over the aggregate halves, over the limit 2^16"""
    n, c = V.shape[0], inputs.site_coords(L)
    na = [L[m] // agg[m] for m in range(4)]
    of = sum((c[:, m] // agg[m]) * int(np.prod(na[:m])) for m in range(4))
    worst, least = 0.0, np.inf
    for i in range(int(np.prod(na))):
        for h in range(2):
            A = V[:, of == i, 2 * h:2 * h + 2].reshape(n, -1).T
            X = np.linalg.inv(np.linalg.qr(A)[1])
            s = n * np.sum(np.linalg.norm(A, axis=0)[:, None] ** 2 * np.abs(X) ** 2) / 65536.0
            worst, least = max(worst, s), min(least, s)
    return least, worst


# every vector a common one plus eps times its own: squared condition about n / eps^2, so the bound on it
# times n is n^2 / eps^2 and crosses 2^16 between eps = 0.2 and 0.05 for 32 vectors
@pytest.mark.parametrize("eps,side", [(0.2, "one"), (0.05, "two"), (1e-3, "two"), (1e-5, "two")])
@pytest.mark.parametrize("vdt", [mrhs.DTYPE_F64, mrhs.DTYPE_F32])
def test_one_pass_rule(eps, side, vdt):
    need_gpu()
    announce("gs one pass eps=%g" % eps)
    L, agg, n = [8, 4, 4, 4], [4, 4, 4, 4], 32
    op = Case(L, 0.3, 341, -0.2).op(agg, agg=agg, prec=mrhs.PREC_F32, short_len=4)
    v = inputs.test_vectors(L, n + 1, 342)
    vn = op.pack(torch.from_numpy(v[:1] + eps * v[1:]), vdt)
    vin = op.unpack(vn, n, vdt).cpu().numpy()
    least, worst = limit_ratio(vin, L, agg)
    assert worst < 1 if side == "one" else least > 1, (least, worst)
    status = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    Q = op.empty(n, mrhs.DTYPE_F32)
    mrhs.block_orthonormalize(op.handle, vn, vdt, Q, mrhs.DTYPE_F32, n, status, op.workspace(n))
    assert int(status.item()) == 0
    # One rounding to FP32 (2^-25) with everything else in FP64: the triangular factor's own error, about
    # 2^-53 n / eps, stays below 4e-10.  One Cholesky pass alone leaves 2^-53 n / eps^2 and more at eps = 1e-5.
    assert per_agg_half_rel(op.unpack(Q, n).cpu().numpy(), oracle.block_gs(L, agg, vin), L, agg) < 2e-7
    op.close()
