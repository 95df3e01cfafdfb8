"""The sizes at which the residual norms refuse a call do not depend on the tile that few vectors take."""
import pytest
import torch

from gpu_helpers import announce, need_gpu
from paper_1601_03184_amd import mrhs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 4, 8])
def test_scratch_and_workspace_limits(n):
    need_gpu()
    L = [32, 32, 24, 12]          # one site per block: 294912 blocks x 8 x 16 bytes are more than 32 MiB
    announce("residual limits n=%d" % n)
    links = torch.eye(3, dtype=torch.complex128, device="cuda").expand(4, 32 * 32 * 24 * 12, 3, 3).contiguous()
    op = mrhs.Operator(L, [1, 1, 1, 1], [4, 4, 4, 4], links, -0.1, 1.0, prec=mrhs.PREC_F32, short_len=4)
    x, b = op.empty(n), op.empty(n)
    x.zero_()
    b.fill_(1.0)
    out = torch.full((n,), float("nan"), dtype=torch.float64, device="cuda")
    with pytest.raises(mrhs.MrhsError) as e:
        mrhs.mrhs_residual_norms_noalloc(op.handle, b, x, n, out)
    assert e.value.code == mrhs.MRHS_EUNSUPPORTED
    least = 294912 * 8 * 16
    ws = torch.empty(least, dtype=torch.uint8, device="cuda")
    with pytest.raises(mrhs.MrhsError) as e:
        mrhs.mrhs_residual_norms(op.handle, b, x, n, out, ws[:least - 1])
    assert e.value.code == mrhs.MRHS_EINVAL
    mrhs.mrhs_residual_norms(op.handle, b, x, n, out, ws)
    assert torch.all(out == 1.0)  # x = 0
    op.close()
