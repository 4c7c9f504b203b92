"""Decode attention at the borders of its launch shapes (eight wavefronts per workgroup up to 256 workgroups with more than
four tiles each; with several heads per KV head wavefronts are kept in step up to 512, and not beyond) and of the
queries' fixed-point operands (heads of very different magnitude in one group, an all-zero head, every number of heads
per KV head, one channel far above the others), against the oracle."""
import numpy as np
import pytest
import torch

from paper_2501_15021_amd import binding as akvq
from paper_2501_15021_amd import synth

pytestmark = pytest.mark.gpu
ATTN_TOL = 2e-3


@pytest.fixture(scope="module")
def orc():
    from oracle import pyoracle
    return pyoracle


def _check(orc, B, Hkv, R, G, T, n_split, q_gain=None, seed=431):
    w = synth.small(f"shape{B}_{Hkv}_{R}", B=B, Hq=Hkv * R, Hkv=Hkv, T=T, G=G, n_text_head=6, n_text_tail=5, top_k=4, W=16)
    d = synth.generate(w, seed=seed)
    if q_gain is not None:
        d["q"] = (d["q"].float() * torch.tensor(q_gain)[None, :, None]).half()
    host = {k: v.numpy() for k, v in d.items()}
    oc = orc.OracleCache(B, Hkv, G, (T + 63) // 64 * 64, 64)
    gc = akvq.Cache(B, Hkv, G, (T + 63) // 64 * 64, 64, fill=0)
    oc.select_tsa(host["is_text"])
    oc.quantize_append(host["k"], host["v"], w.clip)
    akvq.select_salient(gc, akvq.MODE_TSA, is_text=d["is_text"].cuda())
    akvq.quantize_append(gc, d["k"].cuda(), d["v"].cuda(), w.clip)
    ref, lse_ref = oc.decode(host["q"], w.sm_scale)
    out, lse = akvq.decode_attention(gc, d["q"].cuda(), w.sm_scale, n_split=n_split)
    out, lse = out.cpu().numpy(), lse.cpu().numpy()
    rel = np.abs(out - ref).max(-1) / np.maximum(np.abs(ref).max(-1), 1e-6)
    assert rel.max() <= ATTN_TOL, f"{rel.max():.3e}"
    # a logit is off by at most U/2 per channel (U <= 2^-18 of the head's largest rotated channel) against the stored row,
    # whose norm is taken as at most twice the original's; twice that for the two-term bfloat16 operands of 16-bit rows
    k_norm = np.linalg.norm(host["k"].astype(np.float64), axis=-1).max(-1).repeat(R, axis=1)
    q_norm = np.linalg.norm(host["q"].astype(np.float64), axis=-1)
    bound = 2 * 2.0 ** -19 * w.sm_scale * q_norm * 2 * k_norm * np.sqrt(128) + 1e-5 * np.maximum(1.0, np.abs(lse_ref))
    assert (np.abs(lse - lse_ref) <= bound).all(), float((np.abs(lse - lse_ref) / bound).max())


# workgroups = B * Hkv * n_split: 256 / 257 (eight wavefronts or four), 512 / 514 (several heads per KV head: kept in step
# or not); tiles per split around the four that eight wavefronts need
@pytest.mark.parametrize("R,G", [(1, 128), (7, 64)])
@pytest.mark.parametrize("B,Hkv,n_split,tiles", [(64, 4, 1, 5), (64, 4, 1, 4), (1, 257, 1, 5), (32, 4, 4, 9), (2, 257, 1, 5),
                                                 (2, 2, 1, 17), (2, 2, 3, 40)])
def test_launch_shapes(orc, R, G, B, Hkv, n_split, tiles):
    _check(orc, B, Hkv, R, G, tiles * (64 if R == 1 else 32) * n_split - 7, n_split)


@pytest.mark.parametrize("G", [64, 128])
@pytest.mark.parametrize("R", [2, 3, 4, 5, 6, 7, 8])
def test_query_magnitudes(orc, R, G):
    gain = [1.0, 0.0, 2.0 ** -10, 8.0, 1.0, 2.0 ** -14, 0.37, 3.0][:R] * 2
    _check(orc, 2, 2, R, G, 300, 2, q_gain=gain)


@pytest.mark.parametrize("G", [64, 128])
def test_query_magnitudes_one_head(orc, G):
    _check(orc, 2, 4, 1, G, 300, 2, q_gain=[1.0, 0.0, 2.0 ** -14, 8.0])


@pytest.mark.parametrize("R,G", [(1, 128), (1, 64), (2, 64), (7, 64), (8, 128)])
@pytest.mark.parametrize("peak", [16.0, 256.0, 4096.0])
def test_one_dominant_query_channel(orc, R, G, peak):
    """Queries that arrive rotated with one channel far above the rest, against keys that are small there and large
    elsewhere.  The code stream takes every channel as an integer of units U = 2^-19 (one head per KV head: 2^-20) times
    the power of two above the largest channel, so a logit carries 128 roundings of at most U / 2 each times the stored
    key's channel, however small the channels are that matter.  With one cached row the log-sum-exp is the logit."""
    B, Hkv = 16, 4
    rng = np.random.default_rng(int(peak) + R)
    k = rng.standard_normal((B, Hkv, 1, 128)).astype(np.float16)
    k[..., :3] *= np.float16(0.02)
    k[..., 40] *= np.float16(8)
    q = rng.standard_normal((B, Hkv * R, 128)).astype(np.float16)
    q[..., 1] = peak
    c = akvq.Cache(B, Hkv, G, 64, 64, fill=0)
    akvq.quantize_append(c, torch.from_numpy(k).cuda(), torch.from_numpy(k).cuda(), 0.8, flags=akvq.K_PREROTATED)
    scale = 128 ** -0.5
    _, lse = akvq.decode_attention(c, torch.from_numpy(q).cuda(), scale, n_split=1, flags=akvq.Q_PREROTATED)
    lse = lse.cpu().numpy()
    worst = 0.0
    for b in range(B):
        for h in range(Hkv * R):
            codes, s16, zero, _ = orc.quantize_row(k[b, h // R, 0], G, 0.8, rotate=False)
            s, z = s16.view(np.float16).astype(np.float64).repeat(G), zero.astype(np.float64).repeat(G)
            stored, q64 = s * (codes - z), q[b, h].astype(np.float64)
            unit = 2.0 ** (-20 if R == 1 else -19) * 2.0 ** (np.floor(np.log2(np.abs(q64).max())) + 1)
            # independent roundings, uniform over a unit: six standard deviations; sm_scale * log2(e) is folded into several
            # heads' queries, whose power of two can then be twice as far from the largest channel
            bound = 6 * (unit if R == 1 else 2 * unit) / 12 ** 0.5 * np.linalg.norm(stored)
            # 32-bit sums of the code and the zero-point part, a few roundings each
            bound += 8 * 2.0 ** -24 * (np.abs(q64) * s * (codes + np.abs(z))).sum()
            worst = max(worst, abs(lse[b, h] / scale - q64 @ stored) / bound)
    assert worst <= 1.0
