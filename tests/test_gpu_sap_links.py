"""The SAP's block links in LDS: tiles 1 and 2 of every precision, with blocks whose links fit beside
the block residual and blocks whose links do not, directions that a block spans, and a batch of both."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import Case, announce, need_gpu, per_rhs_rel
from paper_1601_03184_amd import inputs, mrhs

pytestmark = pytest.mark.gpu

F64, F32, F16 = mrhs.PREC_F64, mrhs.PREC_F32, mrhs.PREC_F32_F16STORE
TOL = {F64: 1e-12, F32: 1e-5, F16: 5e-3}
SHAPES = [
    ([8, 4, 4, 8], [4, 4, 4, 4]),   # fits; y and z spanned by the block
    ([16, 8, 4, 4], [8, 4, 2, 4]),  # uneven extents
    ([8, 8, 4, 4], [8, 8, 2, 2]),   # does not fit
    ([6, 6, 6, 6], [3, 3, 3, 3]),   # 81 sites: idle lanes in the last wavefront
    ([4, 4, 4, 4], [1, 2, 4, 2]),   # one site thick: no link in x
]


def smooth(ops, vs, ns, n_sap, n_mr):
    bs = [op.pack(torch.from_numpy(v)) for op, v in zip(ops, vs)]
    xs = [torch.zeros_like(b) for b in bs]
    if len(ops) == 1:
        ws = torch.empty(mrhs.mrhs_workspace_bytes(ops[0].handle, ns[0]), dtype=torch.uint8, device="cuda")
        mrhs.sap_smooth_mrhs(ops[0].handle, bs[0], xs[0], ns[0], n_sap, n_mr, ws)
    else:
        hs = [op.handle for op in ops]
        ws = torch.empty(mrhs.mrhs_batched_workspace_bytes(hs, ns), dtype=torch.uint8, device="cuda")
        mrhs.sap_smooth_mrhs_batched(hs, bs, xs, ns, n_sap, n_mr, ws)
    return [(op.unpack(b, n).cpu().numpy(), op.unpack(x, n).cpu().numpy()) for op, b, x, n in zip(ops, bs, xs, ns)]


@pytest.mark.parametrize("prec", [F64, F32, F16])
@pytest.mark.parametrize("tile", [1, 2])
def test_sap_links(prec, tile):
    need_gpu()
    ops, vs, refs, cases = [], [], [], []
    for L, block in SHAPES:
        case = Case(L, 0.3, 361, -0.1)
        cases.append(case)
        op = case.op(block, prec=prec, short_len=2)
        mrhs.mrhs_set_tiles(op.handle, tile, 0)
        ops.append(op)
        vs.append(inputs.test_vectors(L, 3, 362))
    alone = []
    for op, v, case, (L, block) in zip(ops, vs, cases, SHAPES):
        announce("sap links L=%s block=%s prec=%d tile=%d" % (L, block, prec, tile))
        b, x = smooth([op], [v], [3], 2, 3)[0]
        assert per_rhs_rel(x, oracle.sap(L, block, case.U, case.A, b, 2, 3)) < TOL[prec]
        alone.append(x)
    # one workgroup shape for all: the largest block's
    for (b, x), a in zip(smooth(ops, vs, [3] * len(ops), 2, 3), alone):
        assert per_rhs_rel(x, a) < TOL[prec]
    for op in ops:
        op.close()
