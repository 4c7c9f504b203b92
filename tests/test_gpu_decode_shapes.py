"""Decode attention at the borders of its launch shapes (eight wavefronts per workgroup up to 256 workgroups with more than
four tiles each, wavefronts kept in step up to 512, neither beyond) and of the queries' fixed-point operands (heads of
very different magnitude in one group, an all-zero head, every number of heads per KV head), against the oracle."""
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


# workgroups = B * Hkv * n_split: 256 / 257 (eight wavefronts or four), 512 / 514 (kept in step or not); tiles per split
# around the four that eight wavefronts need
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
