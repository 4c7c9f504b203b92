"""Who stores the ring rows of an append (wavefronts of their own, the blocks, or the window's blocks alone by the body with the
ring stores) is chosen by how many workgroups each way brings; whichever it is, a unit stores what it stores when its batch
element is appended alone, row by row where that is short."""
import pytest
import torch

from paper_2501_15021_amd import binding as akvq
from test_gpu_window_rows import NAMES, _rows

pytestmark = pytest.mark.gpu


# (units, rows, window, rows appended before): the window's blocks in workgroups of their own (10 blocks with 3 of the window, 13
# with 4, behind rows that leave a block half full); launches of fewer than two workgroups a CU whose blocks store the ring
# (4 blocks, all of the window); two blocks of the window at the upper and past the upper border; an even split of groups
# without a workgroup more
@pytest.mark.parametrize("B,H,T,W,before", [(43, 2, 300, 64, 0), (64, 2, 290, 64, 17), (24, 4, 410, 128, 0), (33, 4, 128, 128, 0),
                                            (40, 2, 100, 192, 0), (100, 2, 97, 128, 40), (103, 5, 64, 64, 0), (26, 10, 64, 64, 0),
                                            (32, 2, 230, 256, 0), (70, 2, 150, 64, 0)])
@pytest.mark.parametrize("tiers,with_rope", [(False, False), (False, True), (True, False), (True, True)])
def test_ring_rows(B, H, T, W, before, tiers, with_rope):
    k, v, rope = _rows(B, H, before + T, 8)
    gen = torch.Generator().manual_seed(T)
    src = torch.randint(0, T, (B, T), generator=gen).to(torch.int32).cuda()
    tier = torch.randint(0, 4, (B, T), generator=gen).to(torch.uint8).cuda()

    def append(b):
        n = len(range(*b.indices(B)))
        c = akvq.Cache(n, H, 128, (before + T + 63) // 64 * 64, 64, fill=0)
        c.sal_idx[:, :, 0] = before + T // 2
        c.counts().fill_(1)
        c.enable_window(W)
        for lo, hi in ((0, before), (before, before + T)):
            if lo == hi:
                continue
            mapped = tiers and lo == before
            akvq.quantize_append_tiered(c, k[b, :, lo:hi].contiguous(), v[b, :, lo:hi].contiguous(), src[b].clone() if mapped else None,
                                        tier[b].clone() if mapped else None, 0.8, 0.95,
                                        rope=tuple(t[lo:hi].contiguous() for t in rope) if with_rope else None)
        return c

    whole = append(slice(0, B))
    for b in (0, 11, B - 1):
        alone = append(slice(b, b + 1))
        for n in NAMES + ["k_sal", "v_sal"]:
            assert torch.equal(getattr(whole, n)[b], getattr(alone, n)[0]), (n, b)
