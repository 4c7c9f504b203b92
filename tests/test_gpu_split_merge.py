"""Merging the KV splits: split counts around the batches the merge kernel requests its partial results in (four
wavefronts; one, two or eight splits each per round), with more splits than tiles (empty splits) among them."""
import pytest
import torch

from paper_2501_15021_amd import binding as akvq
from paper_2501_15021_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,G", [(4, 4, 128), (14, 2, 64)])
def test_any_number_of_splits_gives_the_unsplit_result(Hq, Hkv, G):
    w = synth.small(f"merge{Hq}", B=2, Hq=Hq, Hkv=Hkv, T=2200, G=G, n_text_head=20, n_text_tail=9, top_k=12, W=16)
    d = synth.generate(w, seed=411, device="cuda")
    c = akvq.Cache(w.B, w.Hkv, G, 2240, 64, fill=0)
    akvq.select_salient(c, akvq.MODE_PSA, q_tail=d["q_tail"], k=d["k"], top_k=w.top_k, sm_scale=w.sm_scale)
    akvq.quantize_append(c, d["k"], d["v"], w.clip)
    one, lse_one = akvq.decode_attention(c, d["q"], w.sm_scale, n_split=1, flags=akvq.OUT_ROTATED)
    # Weights are rounded to 16 significant bits relative to a reference that depends on the split: two results differ by
    # at most 2 * 2^-17 of the weighted sum of |v|, i.e. 2^-16 of the largest stored |v| (scale * 3 levels and the zero
    # point: at most 4 * |clipped extreme|); the 32-bit sums of 2200 terms add less than that again.
    bound = 2.0 * 2.0 ** -16 * 4.0 * float(d["v"].float().abs().max()) * 128 ** 0.5
    for n_split in (2, 3, 4, 5, 8, 9, 31, 32, 33, 64, 65, 100):
        out, lse = akvq.decode_attention(c, d["q"], w.sm_scale, n_split=n_split, flags=akvq.OUT_ROTATED)
        assert torch.isfinite(out).all(), n_split
        assert float((out - one).abs().max()) <= bound, n_split
        assert float((lse - lse_one).abs().max()) <= 1e-5 * max(1.0, float(lse_one.abs().max())), n_split
