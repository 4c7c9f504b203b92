"""Text positions at the borders of the two workgroup sizes (rows of up to 8192 positions, longer ones, more rows than one
workgroup per CU holds) and of their rounds, with rows that start at any byte."""
import pytest
import torch

from paper_2501_15021_amd import binding as akvq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,T,share", [(2, 2, 4096, 0.1), (3, 2, 4097, 0.1), (3, 1, 4111, 1.0), (2, 1, 16384, 0.2), (3, 1, 16385, 0.2), (3, 1, 33001, 0.1),
                                         (2, 1, 20000, 0.0), (64, 8, 4100, 0.1), (57, 9, 4100, 0.1), (3, 2, 8192, 0.1), (3, 2, 8193, 0.1), (3, 1, 12289, 1.0),
                                         (32, 8, 8200, 0.1), (257, 1, 8200, 0.1)])
def test_positions(B, H, T, share):
    mask = (torch.rand(B, T, generator=torch.Generator().manual_seed(T)) < share).to(torch.uint8)
    cap = (int(mask.sum(1).max()) + 63) // 64 * 64 or 64
    c = akvq.Cache(B, H, 128, (T + 63) // 64 * 64, cap, fill=0)
    c.sal_idx.fill_(-7)
    akvq.select_salient(c, akvq.MODE_TSA, is_text=mask.cuda())
    torch.cuda.synchronize()
    for b in range(B):
        want = torch.nonzero(mask[b]).flatten().int()
        assert (c.counts()[b] == len(want)).all()
        assert torch.equal(c.sal_idx[b, :, :len(want)].cpu(), want[None].expand(H, -1)) and (c.sal_idx[b, :, len(want):] == -7).all()
