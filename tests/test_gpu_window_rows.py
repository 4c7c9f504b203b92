"""The ring rows of an append, stored by wavefronts of their own in the launch of the blocks or by the blocks, are bit for bit
those that the same rows leave when they are appended one at a time or in ragged pieces, and the blocks do not change."""
import pytest
import torch

from paper_2501_15021_amd import binding as akvq
from paper_2501_15021_amd import synth

pytestmark = pytest.mark.gpu

NAMES = ["k_win", "v_win", "k_codes", "v_codes", "k_meta", "v_meta"]


def _rows(B, H, T, seed):
    d = synth.generate(synth.small("ring", B=B, Hq=H, Hkv=H, T=T, G=128, n_text_head=5, n_text_tail=3, top_k=8, W=16),
                       seed=seed, device="cuda")
    rope = tuple(torch.from_numpy(t).cuda() for t in synth.rope_tables(torch.arange(T).numpy()))
    return d["k"], d["v"], rope


# one block, a ragged one, one workgroup of the window's blocks and several; windows shorter and longer than the append;
# short salient lists and long ones (whose overlay rows follow in a launch of their own)
@pytest.mark.parametrize("B,H,T,G,W,slots", [(1, 1, 32, 128, 64, 64), (2, 3, 45, 64, 64, 64), (1, 2, 131, 128, 64, 128),
                                             (3, 1, 300, 64, 192, 64), (1, 2, 333, 128, 256, 192)])
@pytest.mark.parametrize("with_rope", [False, True])
def test_plain_rows(B, H, T, G, W, slots, with_rope):
    k, v, rope = _rows(B, H, T, 5)
    got = []
    for cuts in ((0, T), (0, *range(1, T, 1), T) if T < 50 else (0, 1, 17, 100, 101, T)):
        c = akvq.Cache(B, H, G, (T + 63) // 64 * 64, slots, fill=0)
        c.sal_idx[:, :, 0] = T // 2
        c.counts().fill_(1)
        c.enable_window(W)
        for a, b in zip(cuts[:-1], cuts[1:]):
            akvq.quantize_append_tiered(c, k[:, :, a:b].contiguous(), v[:, :, a:b].contiguous(), None, None, 0.8, 1.0,
                                        rope=tuple(t[a:b].contiguous() for t in rope) if with_rope else None)
        got.append(c)
    for n in NAMES + ["k_sal", "v_sal"]:
        assert torch.equal(getattr(got[0], n), getattr(got[1], n)), n


# rows of every tier and padding in the window, the rows' order not their source's
@pytest.mark.parametrize("T,n_rows,W", [(64, 64, 64), (90, 141, 64), (200, 333, 128), (150, 480, 512)])
@pytest.mark.parametrize("with_rope", [False, True])
def test_tiered_rows(T, n_rows, W, with_rope):
    B, H, G = 2, 2, 128
    k, v, rope = _rows(B, H, T, 6)
    gen = torch.Generator().manual_seed(n_rows)
    src = torch.randint(0, T, (B, n_rows), generator=gen).to(torch.int32).cuda()
    tier = torch.randint(0, 4, (B, n_rows), generator=gen).to(torch.uint8).cuda()
    got = []
    for cuts in ((0, n_rows), (0, 7, 8, 33, 61, n_rows)):
        c = akvq.Cache(B, H, G, (n_rows + 63) // 64 * 64, 64, fill=0)
        c.counts().zero_()
        c.enable_window(W)
        for a, b in zip(cuts[:-1], cuts[1:]):
            akvq.quantize_append_tiered(c, k, v, src[:, a:b].contiguous(), tier[:, a:b].contiguous(), 0.8, 0.95,
                                        rope=rope if with_rope else None)
        got.append(c)
    for n in NAMES:
        assert torch.equal(getattr(got[0], n), getattr(got[1], n)), n
    no_token = (tier[:, -1] == akvq.TIER_4BIT_FINE) | (tier[:, -1] == akvq.TIER_PAD)
    zero = (got[0].k_win.reshape(B, H, W, 128)[:, :, (n_rows - 1) % W] == 0).all(-1).all(-1)
    assert torch.equal(zero, no_token)


# launches whose blocks store the ring rows themselves (a window of more than a quarter of the blocks, more than two
# workgroups a CU; the last case also in turned orders) against the batch elements alone, which go the other way
@pytest.mark.parametrize("B,H,T,G,W", [(65, 2, 130, 128, 64), (43, 3, 250, 64, 128), (33, 2, 1010, 128, 512), (160, 4, 1010, 128, 512)])
@pytest.mark.parametrize("tiers,with_rope", [(False, False), (False, True), (True, False), (True, True)])
def test_blocks_store_the_ring(B, H, T, G, W, tiers, with_rope):
    k, v, rope = _rows(B, H, T, 7)
    src = tier = None
    if tiers:
        gen = torch.Generator().manual_seed(T)
        src = torch.randint(0, T, (B, T), generator=gen).to(torch.int32).cuda()
        tier = torch.randint(0, 4, (B, T), generator=gen).to(torch.uint8).cuda()

    def append(b):
        c = akvq.Cache(len(range(*b.indices(B))), H, G, (T + 63) // 64 * 64, 64, fill=0)
        c.sal_idx[:, :, 0] = T // 2
        c.counts().fill_(1)
        c.enable_window(W)
        akvq.quantize_append_tiered(c, k[b].contiguous(), v[b].contiguous(), src[b].clone() if tiers else None,
                                    tier[b].clone() if tiers else None, 0.8, 0.95, rope=rope if with_rope else None)
        return c

    whole = append(slice(0, B))
    for b in (0, 7, B - 1):
        alone = append(slice(b, b + 1))
        for n in NAMES + ["k_sal", "v_sal"]:
            assert torch.equal(getattr(whole, n)[b], getattr(alone, n)[0]), (n, b)
