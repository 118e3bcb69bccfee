"""The partials whose sums test_gpu_mlp_reduce.py compares bit for bit are numbers, and nearly all of them count: a
gradient of random weights on random samples has no parameter that is zero by construction."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
NPARAM = 4737


@pytest.mark.parametrize("nblk", [1, 257])
def test_partials_are_finite_and_mostly_nonzero(nblk):
    import torch
    from paper_2411_09364_amd import les
    n = 256 * nblk - 19
    gen = torch.Generator(device="cuda").manual_seed(nblk)
    params = 0.3 * torch.randn(NPARAM, generator=gen, device="cuda")
    x = torch.rand(n, 7, generator=gen, device="cuda")
    t = torch.randn(n, generator=gen, device="cuda")
    ws = torch.full((nblk, NPARAM + 1), float("nan"), device="cuda")
    g = torch.full((NPARAM,), float("nan"), device="cuda")
    loss = torch.full((1,), float("nan"), device="cuda")
    les.les_mlp_grad(torch.cuda.current_stream().cuda_stream, params.data_ptr(), x.data_ptr(), t.data_ptr(), n,
                     ws.data_ptr(), g.data_ptr(), loss.data_ptr())
    torch.cuda.synchronize()
    for a in (ws.cpu().numpy(), g.cpu().numpy()):
        assert np.isfinite(a).all()
        assert np.count_nonzero(a) > 0.9 * a.size
    assert np.isfinite(loss.item()) and loss.item() > 0
