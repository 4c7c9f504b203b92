"""Selection of short prompts in one launch (one query head per KV head, W = 64, up to 768 keys) at the borders of its three
workgroup sizes: masses against binary64 on the operands the call documents, index sets against the top-k of the call's
own masses.  Neighbours that take the general launches (another head ratio, 769 keys, a scale that is not positive, token-level
pivots) are held to the same."""
import math

import pytest
import torch

from paper_2501_15021_amd import binding as akvq
from paper_2501_15021_amd import synth
from test_gpu_select_chunks import _masses

pytestmark = pytest.mark.gpu


def _select(w, d, top_k, mode=akvq.MODE_PSA, sm_scale=None):
    c = akvq.Cache(w.B, w.Hkv, 128, (w.T + 63) // 64 * 64, max(64, (top_k + 63) // 64 * 64), fill=0)
    mass = torch.full((w.B, w.Hkv, w.T), float("nan"), device="cuda")
    akvq.select_salient(c, mode, q_tail=d["q_tail"], k=d["k"], top_k=top_k, sm_scale=w.sm_scale if sm_scale is None else sm_scale,
                        mass_out=mass)
    torch.cuda.synchronize()
    return c, mass


@pytest.mark.parametrize("B,H,T,top_k", [(1, 3, 64, 8), (2, 2, 65, 65), (1, 3, 127, 15), (1, 2, 128, 1), (3, 1, 255, 8), (1, 4, 256, 64),
                                         (1, 4, 257, 8), (2, 2, 320, 128), (1, 2, 511, 32), (1, 2, 512, 200), (1, 2, 513, 16), (1, 4, 640, 8),
                                         (2, 3, 767, 64), (1, 2, 768, 300), (1, 2, 769, 16)])
def test_small_prompts(B, H, T, top_k):
    w = synth.small(f"small{T}", B=B, Hq=H, Hkv=H, T=T, G=128, n_text_head=5, n_text_tail=3, top_k=8, W=64)
    d = synth.generate(w, seed=631, device="cuda")
    c, mass = _select(w, d, top_k)
    want = _masses(d, w)
    # the bar of the pivot score: 4e-5 of the element (32-bit sums and exponentials), 1e-12 absolute
    assert ((mass.double() - want).abs() <= 4e-5 * want + 1e-12).all()
    k = min(top_k, T)
    order = torch.sort(mass, dim=-1, descending=True, stable=True).indices[..., :k].sort(-1).values
    assert torch.equal(c.sal_idx[..., :k].long(), order) and (c.counts() == k).all()
    # the masses added over the heads are scored by the general launches: the same up to the order of the sums
    shared, mass2 = _select(w, d, top_k, mode=akvq.MODE_PSA_SHARED)
    assert ((mass2.double() - want).abs() <= 4e-5 * want + 1e-12).all()
    assert (shared.counts() == k).all()


@pytest.mark.parametrize("fill", [0.0, 1.0])
def test_equal_masses(fill):
    """Every key the same: a scale of 0 goes through the general launches, constant keys through the one launch; the causal
    edge leaves the first T - 63 masses equal and the lowest positions win."""
    T = 600
    w = synth.small("flat", B=1, Hq=2, Hkv=2, T=T, G=128, n_text_head=5, n_text_tail=3, top_k=8, W=64)
    d = synth.generate(w, seed=633, device="cuda")
    d["k"] = torch.full_like(d["k"], fill)
    for scale in (w.sm_scale, 0.0):
        c, mass = _select(w, d, 16, sm_scale=scale)
        want = sum(1.0 / (T - 63 + i) for i in range(64))
        assert torch.allclose(mass[..., : T - 63].double(), torch.full_like(mass[..., : T - 63], want).double(), rtol=1e-5, atol=0)
        assert math.isclose(float(mass.double().sum()), 2 * 64, rel_tol=1e-5)
        order = torch.sort(mass, dim=-1, descending=True, stable=True).indices[..., :16].sort(-1).values
        assert torch.equal(c.sal_idx[..., :16].long(), order)


@pytest.mark.parametrize("T", [256, 512, 768])
def test_one_key_far_above_the_rest(T):
    """One key about 200 nats above all others, in each of the last sixteen places of a wavefront's 64 keys (one per head) and
    in every wavefront: an exponent against a reference that misses it would overflow.  Its mass is that of the rows that see
    it, the others' are below binary32; the rows that don't see it are the softmax of the rest, to the bar above."""
    w = synth.small("spike", B=T // 64, Hq=16, Hkv=16, T=T, G=128, n_text_head=5, n_text_tail=3, top_k=8, W=64)
    gen = torch.Generator(device="cuda").manual_seed(637)
    # normal values, so that the other logits are within 10 nats of 0 (a generated prompt has rows whose own outliers reach
    # 200 nats: one of 64 rows then has its mass elsewhere): the others' share is below 768 * exp(-190)
    d = {n: torch.randn(w.B, 16, rows, 128, generator=gen, device="cuda").half() for n, rows in (("q_tail", 64), ("k", T))}
    d["q_tail"][..., 0] = 4.0
    d["k"][..., 0] = 0.0
    at = 64 * torch.arange(w.B)[:, None] + 48 + torch.arange(16)[None, :]
    for b in range(w.B):
        for h in range(16):
            d["k"][b, h, at[b, h]] = 0.0
            d["k"][b, h, at[b, h], 0] = 200.0 / (4.0 * w.sm_scale)
    c, mass = _select(w, d, 1)
    want = _masses(d, w)
    assert torch.isfinite(mass).all()
    assert ((mass.double() - want).abs() <= 4e-5 * want + 1e-12).all()
    order = torch.sort(mass, dim=-1, descending=True, stable=True).indices[..., :1]
    assert torch.equal(c.sal_idx[..., :1].long(), order)
    early = at < T - 64
    assert torch.equal(c.sal_idx[..., 0].cpu().long()[early], at[early])
    spike = mass.cpu().gather(-1, at[..., None])[..., 0]
    assert ((spike - 64.0).abs() <= 64 * 4e-5)[early].all()
