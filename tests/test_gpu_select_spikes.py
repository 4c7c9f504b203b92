"""Chunks of 2048 keys whose exponentials are added up without a look at the logits: single keys far above their row's reference,
in every place of a block of 64 keys, by less and by more than what binary32 holds, and keys far below it."""
import pytest
import torch

from paper_2501_15021_amd import binding as akvq
from paper_2501_15021_amd import synth
from test_gpu_select_chunks import _masses

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv", [(14, 2), (8, 1), (2, 1)])
@pytest.mark.parametrize("nats", [30.0, 60.0, 200.0, -200.0])
def test_keys_far_above_the_rest(Hq, Hkv, nats):
    T, B = 4200, 576 // Hkv  # three chunks: more than two workgroups per CU, so none is shorter
    w = synth.small("spikes", B=B, Hq=Hq, Hkv=Hkv, T=T, G=128, n_text_head=5, n_text_tail=3, top_k=8, W=64)
    gen = torch.Generator(device="cuda").manual_seed(641)
    d = {n: torch.randn(B, H, rows, 128, generator=gen, device="cuda").half() for n, H, rows in (("q_tail", Hq, 64), ("k", Hkv, T))}
    d["q_tail"][..., 0] = 4.0
    d["k"][..., 0] = 0.0
    units = torch.arange(B * Hkv, device="cuda").reshape(B, Hkv)
    at = (7 * units + 64 * (units % 61)) % (T - 64)  # any place of a block, first and later blocks of all chunks
    spike = torch.zeros(128, device="cuda")
    spike[0] = nats / (4.0 * w.sm_scale)
    d["k"].scatter_(2, at[..., None, None].expand(-1, -1, 1, 128), spike.half().expand(B, Hkv, 1, 128))
    c = akvq.Cache(B, Hkv, 128, 4224, 64, fill=0)
    mass = torch.full((B, Hkv, T), float("nan"), device="cuda")
    akvq.select_salient(c, akvq.MODE_PSA, q_tail=d["q_tail"], k=d["k"], top_k=8, sm_scale=w.sm_scale, mass_out=mass)
    torch.cuda.synchronize()
    want = _masses(d, w)
    # the bar of the pivot score: 4e-5 of the element (32-bit sums and exponentials), 1e-12 absolute
    assert ((mass.double() - want).abs() <= 4e-5 * want + 1e-12).all()
    order = torch.sort(mass, dim=-1, descending=True, stable=True).indices[..., :8].sort(-1).values
    assert torch.equal(c.sal_idx[..., :8].long(), order)
