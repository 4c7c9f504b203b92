"""Pivot scoring at the borders of its chunks: the keys a workgroup scores shrink from 2048 to 128 for small problems, and
a workspace that only holds the statistics of 2048-key chunks is still served.  Masses against binary64 on the operands
the call documents (rounded to bfloat16), index sets against the top-k of the call's own masses."""
import ctypes as C
import math

import pytest
import torch

from paper_2501_15021_amd import binding as akvq
from paper_2501_15021_amd import synth

pytestmark = pytest.mark.gpu


def _masses(d, w):
    R = w.Hq // w.Hkv
    hidden = torch.arange(w.T, device="cuda")[None, :] > (w.T - w.W + torch.arange(w.W, device="cuda"))[:, None]
    mass = torch.empty(w.B, w.Hkv, w.T, dtype=torch.float64, device="cuda")
    for b in range(w.B):
        for h in range(w.Hkv):
            q = d["q_tail"][b, h * R:(h + 1) * R].bfloat16().double()
            s = torch.matmul(q, d["k"][b, h].bfloat16().double().t().contiguous()) * w.sm_scale
            mass[b, h] = torch.softmax(s.masked_fill(hidden, -math.inf), dim=-1).sum(dim=(0, 1))
    return mass


# (B, Hq, Hkv, T): one chunk up to 64 of them, of 64 to 2048 keys, the tail rows across one to three chunks, one to eight
# query heads per KV head, the shortest context
@pytest.mark.parametrize("B,Hq,Hkv,T", [(1, 4, 4, 64), (1, 4, 4, 129), (1, 4, 4, 256), (2, 8, 4, 385), (1, 14, 2, 2048 + 1),
                                        (1, 8, 1, 1000), (4, 32, 32, 1300), (2, 64, 64, 4100), (1, 7, 1, 9000),
                                        (1, 4, 2, 16500)])
def test_chunk_sizes(B, Hq, Hkv, T):
    w = synth.small(f"chunk{T}", B=B, Hq=Hq, Hkv=Hkv, T=T, G=128, n_text_head=5, n_text_tail=3, top_k=8, W=64)
    d = synth.generate(w, seed=521, device="cuda")
    want = _masses(d, w)
    L = akvq.lib()
    c = akvq.Cache(B, Hkv, 128, (T + 63) // 64 * 64, 64, fill=0)
    fine = L.akvq_select_workspace_bytes(B, Hq, Hkv, T, 64)
    up = lambda n: (n + 255) // 256 * 256  # noqa: E731
    coarse = up(B * Hq * ((T + 2047) // 2048) * 64 * 8) + up(B * Hkv * T * 4) + up(B * T * 4)
    assert fine >= coarse
    for nbytes in sorted({fine, coarse}):
        ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")
        mass = torch.full((B, Hkv, T), float("nan"), device="cuda")
        s = c.struct()
        args = (C.byref(s), akvq.MODE_PSA, None, d["q_tail"].data_ptr(), Hq, d["k"].data_ptr(), T, 64, w.top_k, w.sm_scale,
                mass.data_ptr(), ws.data_ptr())
        stream = torch.cuda.current_stream().cuda_stream
        assert L.akvq_select_salient(*args, coarse - 1, stream) == -4  # what was too small stays too small
        assert L.akvq_select_salient(*args, nbytes, stream) == 0
        torch.cuda.synchronize()
        # the bar of the pivot score: 4e-5 of the element (32-bit sums and exponentials), 1e-12 absolute
        assert ((mass.double() - want).abs() <= 4e-5 * want + 1e-12).all(), nbytes
        order = torch.sort(mass, dim=-1, descending=True, stable=True).indices[..., :w.top_k].sort(-1).values
        assert torch.equal(c.sal_idx[..., :w.top_k].long(), order), nbytes


@pytest.mark.parametrize("B,Hq,Hkv,T,longest", [(1, 28, 4, 16384, 16400), (1, 4, 4, 4096, 40000), (3, 8, 4, 1000, 2500)])
def test_workspace_of_a_longer_prompt(B, Hq, Hkv, T, longest):
    """One workspace sized for the longest prompt scores a shorter one in the chunks of its own size (same bits), and each
    smaller workspace down to that of 2048-key chunks in the finest ones that fit, up to the order of the sums."""
    w = synth.small(f"longer{T}", B=B, Hq=Hq, Hkv=Hkv, T=T, G=128, n_text_head=5, n_text_tail=3, top_k=8, W=64)
    d = synth.generate(w, seed=523, device="cuda")
    want = _masses(d, w)
    L = akvq.lib()
    c = akvq.Cache(B, Hkv, 128, (T + 63) // 64 * 64, 64, fill=0)
    s = c.struct()
    up = lambda n: (n + 255) // 256 * 256  # noqa: E731

    def masses(nbytes):
        ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")
        mass = torch.full((B, Hkv, T), float("nan"), device="cuda")
        st = L.akvq_select_salient(C.byref(s), akvq.MODE_PSA, None, d["q_tail"].data_ptr(), Hq, d["k"].data_ptr(), T, 64,
                                   w.top_k, w.sm_scale, mass.data_ptr(), ws.data_ptr(), nbytes,
                                   torch.cuda.current_stream().cuda_stream)
        assert st == 0
        torch.cuda.synchronize()
        assert ((mass.double() - want).abs() <= 4e-5 * want + 1e-12).all(), nbytes
        return mass

    own = masses(L.akvq_select_workspace_bytes(B, Hq, Hkv, T, 64))
    assert torch.equal(masses(L.akvq_select_workspace_bytes(B, Hq, Hkv, longest, 64)), own)
    rest = up(B * Hkv * T * 4) + up(B * T * 4)
    for chunk in (128, 256, 512, 1024, 2048):
        masses(up(B * Hq * ((T + chunk - 1) // chunk) * 64 * 8) + rest)


# as many units as leave the last of two, three and four chunks short, or fill the CUs with one chunk each
@pytest.mark.parametrize("B,Hq,Hkv,T", [(23, 32, 8, 258), (13, 32, 32, 734), (40, 28, 4, 1300), (43, 12, 6, 2049), (5, 64, 8, 3001),
                                        (30, 12, 2, 2900), (3, 40, 5, 6000), (64, 8, 8, 640)])
def test_equal_chunks(B, Hq, Hkv, T):
    test_chunk_sizes(B, Hq, Hkv, T)
