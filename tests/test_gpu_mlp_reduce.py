"""The sum of the training gradient's block partials at the edges of its row chunks (256 rows): bit for bit the
float32 sums in block order of the partials that the call leaves in its workspace."""
import numpy as np
import pytest

from tests.cases import say

pytestmark = pytest.mark.gpu
NPARAM = 4737


# one block, a part of a chunk, a whole one, one row more, several chunks, the most blocks (1024)
@pytest.mark.parametrize("nblk", [1, 3, 255, 256, 257, 769, 1024])
def test_partials_are_summed_in_block_order(nblk):
    import torch
    from paper_2411_09364_amd import les
    n = 256 * nblk - 19
    say(f"mlp gradient partials: {nblk} blocks")
    gen = torch.Generator(device="cuda").manual_seed(nblk)
    params = 0.3 * torch.randn(NPARAM, generator=gen, device="cuda")
    x = torch.rand(n, 7, generator=gen, device="cuda")
    t = torch.randn(n, generator=gen, device="cuda")
    assert les.les_mlp_workspace_bytes(n) == nblk * (NPARAM + 1) * 4
    ws = torch.empty(nblk, NPARAM + 1, device="cuda")
    g = torch.full((NPARAM,), float("nan"), device="cuda")
    loss = torch.full((1,), float("nan"), device="cuda")
    les.les_mlp_grad(torch.cuda.current_stream().cuda_stream, params.data_ptr(), x.data_ptr(), t.data_ptr(), n,
                     ws.data_ptr(), g.data_ptr(), loss.data_ptr())
    torch.cuda.synchronize()
    s = np.zeros(NPARAM + 1, dtype=np.float32)
    for row in ws.cpu().numpy():
        s = s + row
    assert np.abs(s).min() >= 0 and np.abs(s[:NPARAM]).max() > 0
    assert np.array_equal(g.cpu().numpy(), s[:NPARAM])
    assert loss.item() == s[NPARAM] / np.float32(n)
