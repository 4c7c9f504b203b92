"""Appends of more workgroups than the card holds at once, and of so many that their units' orders are turned: what a unit
stores is bit for bit what the same rows store when its batch element is appended alone, in a launch small enough to keep the
plain order."""
import pytest
import torch

from paper_2501_15021_amd import binding as akvq

pytestmark = pytest.mark.gpu


# an even number of workgroups a unit (8, 10, 20: with a ragged last block, with units that don't fill a cycle of eight),
# and the same with an odd number, which is not turned; from 10240 workgroups on turned (8, 10, 20 a unit; 9: not)
@pytest.mark.parametrize("B,H,T,G,before", [(80, 8, 1024, 128, 0), (103, 5, 1207, 64, 0), (37, 7, 2500, 128, 61), (72, 8, 1121, 128, 0),
                                            (9, 8, 1024, 128, 0), (13, 5, 1207, 64, 0), (5, 7, 2500, 128, 61),
                                            (9, 8, 1121, 128, 0)])
def test_unit_order(B, H, T, G, before):
    gen = torch.Generator(device="cuda").manual_seed(T)
    k, v = (torch.randn(B, H, T, 128, generator=gen, device="cuda", dtype=torch.float16) for _ in range(2))

    def append(k, v):
        c = akvq.Cache(k.shape[0], H, G, (before + T + 63) // 64 * 64, 64, fill=0)
        c.sal_idx[:, :, 0] = before + T // 3
        c.counts().fill_(1)
        if before:
            akvq.quantize_append(c, k[:, :, :before].contiguous(), v[:, :, :before].contiguous(), 0.8)
        akvq.quantize_append(c, k, v, 0.8)
        return c

    whole = append(k, v)
    for b in range(B) if B < 20 else (0, 1, 6, 7, 8, 21, B - 1):
        alone = append(k[b:b + 1].contiguous(), v[b:b + 1].contiguous())
        for n in ("k_codes", "v_codes", "k_meta", "v_meta", "k_sal", "v_sal"):
            assert torch.equal(getattr(whole, n)[b], getattr(alone, n)[0]), (n, b)
