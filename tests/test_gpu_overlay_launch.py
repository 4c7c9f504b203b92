"""Long salient lists, whose 16-bit V rows are stored by overlay tiles in the launch of the blocks: bit for bit what short
lists store, where the block kernel writes every row itself (64 slots of the list at a time)."""
import pytest
import torch

from paper_2501_15021_amd import binding as akvq
from paper_2501_15021_amd import synth

pytestmark = pytest.mark.gpu


def _append(k, v, G, rows, slots, rope, cuts):
    B, H, T, _ = k.shape
    c = akvq.Cache(B, H, G, (T + 63) // 64 * 64, slots, fill=0)
    c.sal_idx[:, :, : len(rows)] = torch.tensor(rows, dtype=torch.int32, device="cuda")
    c.counts().fill_(len(rows))
    for a, b in zip(cuts[:-1], cuts[1:]):
        part = [x[:, :, a:b].contiguous() for x in (k, v)]
        if rope is None:
            akvq.quantize_append(c, *part, 0.8)
        else:
            akvq.quantize_append_tiered(c, *part, None, None, 0.8, 1.0, rope=tuple(t[a:b].contiguous() for t in rope))
    return c


# capacities of one to four workgroups of overlay tiles (an odd number of them leaves one half of the launch without), full
# and ragged lists, blocks that end inside a workgroup; pieces that split an overlay tile
@pytest.mark.parametrize("B,H,T,G,slots,n,pieces", [(1, 1, 128, 128, 128, 128, ()), (2, 3, 200, 64, 128, 97, ()), (1, 2, 333, 128, 192, 129, (31, 34)),
                                                    (3, 1, 500, 64, 320, 300, (257,)), (1, 4, 1000, 128, 576, 513, (32, 96, 500))])
@pytest.mark.parametrize("with_rope", [False, True])
def test_overlay_rows(B, H, T, G, slots, n, pieces, with_rope):
    d = synth.generate(synth.small("ovl", B=B, Hq=H, Hkv=H, T=T, G=G, n_text_head=5, n_text_tail=3, top_k=8, W=16), seed=91,
                       device="cuda")
    rope = tuple(torch.from_numpy(t).cuda() for t in synth.rope_tables(torch.arange(T).numpy())) if with_rope else None
    rows = sorted(torch.randperm(T, generator=torch.Generator().manual_seed(n))[:n].tolist())
    long = _append(d["k"], d["v"], G, rows, slots, rope, (0, *pieces, T))
    for s in range(0, n, 64):
        short = _append(d["k"], d["v"], G, rows[s:s + 64], 64, rope, (0, T))
        m = len(rows[s:s + 64])
        assert torch.equal(long.k_sal[:, :, s:s + m], short.k_sal[:, :, :m])
        for tile in range((m + 31) // 32):
            assert torch.equal(long.v_sal[:, :, s // 32 + tile], short.v_sal[:, :, tile]), (s, tile)
        assert torch.equal(long.k_codes, short.k_codes) and torch.equal(long.v_codes, short.v_codes)


# many units, against batch elements appended alone (few units: no idle workgroup, one launch): an idle workgroup a unit (four and
# six without it), behind rows that leave a block half full, and one or two blocks whose overlay goes out in a second launch
@pytest.mark.parametrize("B,H,T,slots,before", [(65, 2, 80, 576, 17), (43, 6, 300, 1152, 0), (256, 2, 40, 128, 0), (103, 5, 9, 192, 50),
                                                (60, 5, 100, 256, 30)])
@pytest.mark.parametrize("with_rope", [False, True])
def test_overlay_of_many_units(B, H, T, slots, before, with_rope):
    n = before + T
    d = synth.generate(synth.small("ovm", B=B, Hq=H, Hkv=H, T=n, G=128, n_text_head=5, n_text_tail=3, top_k=8, W=16 if n < 64 else 64), seed=93,
                       device="cuda")
    rope = tuple(torch.from_numpy(t).cuda() for t in synth.rope_tables(torch.arange(n).numpy())) if with_rope else None
    rows = sorted(torch.randperm(n, generator=torch.Generator().manual_seed(n))[:min(slots, n)].tolist())
    cuts = (0, before, n) if before else (0, n)
    whole = _append(d["k"], d["v"], 128, rows, slots, rope, cuts)
    for b in (0, 7, B - 1):
        alone = _append(d["k"][b:b + 1], d["v"][b:b + 1], 128, rows, slots, rope, cuts)
        for name in ("k_sal", "v_sal", "k_codes", "v_codes", "k_meta", "v_meta"):
            assert torch.equal(getattr(whole, name)[b], getattr(alone, name)[0]), (name, b)
