"""Salient lists of more than 2048 entries, whose run of a block is found by sampling a stretch of the list again: bit for bit
what the lists of at most 2048 entries that make them up store."""
import pytest
import torch

from paper_2501_15021_amd import synth
from test_gpu_overlay_launch import _append

pytestmark = pytest.mark.gpu


# one sample more than 32 entries apart, up to 96 (two loads cover a stretch) and beyond (sampled again, once and twice more);
# dense lists (whole blocks salient), scattered ones, and one that starts late
@pytest.mark.parametrize("T,n,late", [(2100, 2049, 0), (9000, 2049, 6800), (9000, 4097, 0), (6200, 6144, 0), (9000, 6145, 0), (30000, 12000, 0)])
def test_long_lists(T, n, late):
    B, H, slots = 1, 2, (n + 63) // 64 * 64
    d = synth.generate(synth.small("list", B=B, Hq=H, Hkv=H, T=T, G=128, n_text_head=5, n_text_tail=3, top_k=8, W=16), seed=95, device="cuda")
    rows = sorted((late + torch.randperm(T - late, generator=torch.Generator().manual_seed(n))[:n]).tolist())
    long = _append(d["k"], d["v"], 128, rows, slots, None, (0, T))
    # (marked salient: all of them, and no other row)
    for s in range(0, n, 2048):
        part = rows[s:s + 2048]
        short = _append(d["k"], d["v"], 128, part, 2048, None, (0, T))
        assert torch.equal(long.k_sal[:, :, s:s + len(part)], short.k_sal[:, :, :len(part)]), s
        tiles = (len(part) + 31) // 32
        assert torch.equal(long.v_sal[:, :, s // 32: s // 32 + tiles], short.v_sal[:, :, :tiles]), s
        assert torch.equal(long.k_codes, short.k_codes) and torch.equal(long.v_codes, short.v_codes)
    salient = torch.zeros(long.k_meta.numel() // (B * H), dtype=torch.bool)
    salient[torch.tensor(rows)] = True
    marked = (long.k_meta.view(torch.int32).reshape(B * H, -1) & 0x8000) != 0
    assert torch.equal(marked.cpu(), salient[None].expand(B * H, -1))
