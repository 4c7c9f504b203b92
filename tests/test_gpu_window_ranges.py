"""Windowed appends whose blocks go out in one launch (few workgroups) or in two: the stored bytes, rings included, are the
same as those of the same rows appended for every batch element alone, and the plain planes those of an append without
a window."""
import pytest
import torch

from paper_2501_15021_amd import binding as akvq
from paper_2501_15021_amd import synth

pytestmark = pytest.mark.gpu


def _append(k, v, W, before):
    B, H, T, _ = k.shape
    c = akvq.Cache(B, H, 128, (before + T + 63) // 64 * 64, 64, fill=0)
    c.sal_idx[:, :, 0] = before + T // 2
    c.sal_idx[:, :, 1] = before + T - 1
    c.counts().fill_(2)
    if W:
        c.enable_window(W)
    if before:
        akvq.quantize_append_tiered(c, k[:, :, :before].contiguous(), v[:, :, :before].contiguous(), None, None, 0.8, 1.0)
    akvq.quantize_append_tiered(c, k, v, None, None, 0.8, 1.0)
    names = ["k_codes", "v_codes", "k_meta", "v_meta", "k_sal", "v_sal"] + (["k_win", "v_win"] if W else [])
    return {n: getattr(c, n) for n in names}


# (B, heads, rows, window, rows in the cache before): launches of up to 112 and of more than 1024 workgroups; no block, one
# block and several in front of the window; a window longer than the append; an odd start inside a block
@pytest.mark.parametrize("B,H,T,W,before", [(16, 8, 512, 64, 0), (16, 8, 545, 64, 0), (33, 8, 130, 64, 0), (3, 4, 63, 64, 0),
                                            (3, 4, 97, 64, 0), (2, 4, 700, 128, 33), (40, 8, 300, 128, 17)])
def test_window_ranges(B, H, T, W, before):
    d = synth.generate(synth.small("win", B=B, Hq=H, Hkv=H, T=T, G=128, n_text_head=5, n_text_tail=3, top_k=8, W=16),
                       seed=77, device="cuda")
    k, v = d["k"], d["v"]
    whole, plain = _append(k, v, W, before), _append(k, v, 0, before)
    for n, t in plain.items():
        assert torch.equal(whole[n], t), n
    for b in sorted({0, B // 2, B - 1}):
        alone = _append(k[b:b + 1].contiguous(), v[b:b + 1].contiguous(), W, before)
        for n, t in alone.items():
            assert torch.equal(whole[n][b:b + 1], t), (n, b)


# workgroups of the append as one launch (four blocks each, window blocks apart from the others, K and V): the most that one
# launch takes, one group more, and the same with an odd start and a window that starts inside a block
@pytest.mark.parametrize("B,H,T,W,before,groups", [(16, 8, 416, 64, 0, 1024), (16, 8, 448, 64, 0, 1024), (16, 8, 480, 64, 0, 1280),
                                                   (64, 8, 60, 64, 33, 1024), (32, 8, 250, 64, 37, 1536), (32, 8, 150, 64, 37, 1024),
                                                   (8, 16, 390, 128, 5, 1024), (8, 16, 500, 128, 5, 1280)])
def test_at_the_largest_single_launch(B, H, T, W, before, groups):
    first, end = before // 32, (before + T + 31) // 32
    window_first = max(before + T - W, before) // 32
    assert ((window_first - first + 3) // 4 + (end - window_first + 3) // 4) * 2 * B * H == groups
    test_window_ranges(B, H, T, W, before)
