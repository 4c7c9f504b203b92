"""Appends whose groups of four blocks run on from unit to unit (many units, a twelfth of the wavefronts idle otherwise), bit
for bit against batch elements appended alone (few units: groups of their own)."""
import pytest
import torch

from paper_2501_15021_amd import binding as akvq
from paper_2501_15021_amd import synth

pytestmark = pytest.mark.gpu


def _append(d, b, G, clip, before, rope, tiers):
    k, v = d["k"][b].clone(), d["v"][b].clone()
    B, H, T, _ = k.shape
    rows = T if tiers is None else tiers[0].shape[1]
    c = akvq.Cache(B, H, G, (before + rows + 63) // 64 * 64, 64, fill=0)
    c.sal_idx[:, :, :3] = torch.tensor([0, before + 1, before + rows - 1], dtype=torch.int32, device="cuda")
    c.counts().fill_(3)
    c.T_len = before
    if tiers is not None:
        akvq.quantize_append_tiered(c, k, v, tiers[0][b].clone(), tiers[1][b].clone(), clip, 1.0, rope=rope)
    elif rope is not None:
        akvq.quantize_append_tiered(c, k, v, None, None, clip, 1.0, rope=rope)
    else:
        akvq.quantize_append(c, k, v, clip)
    return c


# two to 33 blocks, the number of units no multiple of four (a group that ends behind the last block), rows that leave the first
# block partly old, just above two, five and ten workgroups per CU.  The last two keep their own groups: two workgroups per CU, and
# no round of workgroups saved (test_append_runs.py says which kernel each takes)
FLAT = [(257, 1, 33, 128, 0), (67, 4, 70, 64, 0), (67, 2, 140, 128, 17), (43, 3, 200, 64, 5), (33, 2, 400, 128, 0), (23, 2, 640, 128, 31), (15, 2, 1040, 64, 0),
        (131, 1, 150, 128, 0), (259, 1, 33, 128, 0), (81, 2, 400, 128, 5), (161, 1, 919, 128, 0)]
OWN_GROUPS = [(128, 2, 30, 128, 9), (60, 2, 270, 128, 0)]


def rows_and_plan(B, T, before, kind):
    """(old rows, new rows, row plan) of a case."""
    if kind != "tiers":
        return before, T, None
    text = synth.is_text_mask(synth.small("flat", B=B, Hq=1, Hkv=1, T=T, G=128, n_text_head=5, n_text_tail=3, top_k=8, W=16))
    src, tier, _ = synth.tiered_rows(text[None].repeat(B, 0), [[1]] * B)
    return before + before % 2, src.shape[1], (src, tier)  # (a pair starts on an even row)


@pytest.mark.parametrize("B,H,T,G,before", FLAT + OWN_GROUPS)
@pytest.mark.parametrize("kind", ["plain", "rope", "tiers"])
def test_flat_groups(B, H, T, G, before, kind):
    d = synth.generate(synth.small("flat", B=B, Hq=H, Hkv=H, T=T, G=G, n_text_head=5, n_text_tail=3, top_k=8, W=16), seed=97, device="cuda")
    rope = tuple(torch.from_numpy(t).cuda() for t in synth.rope_tables(torch.arange(T).numpy())) if kind != "plain" else None
    before, _, plan = rows_and_plan(B, T, before, kind)
    tiers = None if plan is None else tuple(torch.from_numpy(x).cuda() for x in plan)
    whole = _append(d, slice(None), G, 0.8, before, rope, tiers)
    for b in (0, B // 2, B - 1):
        alone = _append(d, slice(b, b + 1), G, 0.8, before, rope, tiers)
        for name in ("k_codes", "v_codes", "k_meta", "v_meta", "k_sal", "v_sal"):
            assert torch.equal(getattr(whole, name)[b], getattr(alone, name)[0]), (name, b)
        if whole.fine_mask is not None:
            assert torch.equal(whole.fine_mask[b], alone.fine_mask[0])
