"""Pivot scoring that reads every key once, W = 64: one workgroup per query head (short prompts) or several that exchange their
row statistics.  Masses against binary64 on the operands the call documents, index sets against the top-k of the call's
own masses, at the borders of the rule that chooses it (score_path), of its chunks of 512 keys and of its rounds of heads."""
import ctypes as C

import pytest
import torch

from paper_2501_15021_amd import binding as akvq
from paper_2501_15021_amd import synth
from paper_2501_15021_amd.build import NOWAIT
from test_gpu_select_chunks import _masses

pytestmark = pytest.mark.gpu


def _inputs(B, Hq, Hkv, T, seed=811):
    w = synth.small(f"once{T}", B=B, Hq=Hq, Hkv=Hkv, T=T, G=128, n_text_head=5, n_text_tail=3, top_k=8, W=64)
    return w, synth.generate(w, seed=seed, device="cuda")


def _select(w, d, top_k=8, lib=None, nbytes=None, mode=akvq.MODE_PSA):
    L = lib or akvq.lib()
    nbytes = akvq.lib().akvq_select_workspace_bytes(w.B, w.Hq, w.Hkv, w.T, 64) if nbytes is None else nbytes
    c = akvq.Cache(w.B, w.Hkv, 128, (w.T + 63) // 64 * 64, 64, fill=0)
    ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")  # stale words that look published
    mass = torch.full((w.B, w.Hkv, w.T), float("nan"), device="cuda")
    s = c.struct()
    st = L.akvq_select_salient(C.byref(s), mode, None, C.c_void_p(d["q_tail"].data_ptr()), w.Hq, C.c_void_p(d["k"].data_ptr()),
                               w.T, 64, top_k, C.c_float(w.sm_scale), C.c_void_p(mass.data_ptr()), C.c_void_p(ws.data_ptr()),
                               C.c_size_t(nbytes), C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == 0
    torch.cuda.synchronize()
    return c, mass


def _check(w, d, c, mass, top_k=8):
    want = _masses(d, w)
    # the bar of the pivot score: 4e-5 of the element (32-bit sums and exponentials), 1e-12 absolute
    # (the smallest ones': their logits lie up to 450 below the row's reference, base 2, and are rounded there: 1.9e-5)
    assert ((mass.double() - want).abs() <= 4e-5 * want + 1e-12).all()
    # ... and of all together, which are those near the reference: about twenty roundings of 2^-24 (an exponential, the row's sums,
    # the division, the column's sums over rows and heads); 3e-8 to 5e-7 here
    assert (mass.double() - want).norm() <= 1.2e-6 * want.norm()
    order = torch.sort(mass, dim=-1, descending=True, stable=True).indices[..., :top_k].sort(-1).values
    assert torch.equal(c.sal_idx[..., :top_k].long(), order) and (c.counts() == top_k).all()


# one head per KV head: 512 workgroups of the small kernel and one more head, two chunks and two tokens more, a last chunk of one
# key, 64 workgroups of up to four chunks (two passes) and more, heads in one round and in several, 32 and 33 chunks (one and two
# batches of words), 64 and the first prompt beyond
@pytest.mark.parametrize("B,H,T", [(16, 32, 513), (19, 27, 513), (19, 27, 768), (11, 3, 769), (17, 2, 1024), (11, 2, 1025), (9, 2, 1537), (5, 40, 1500),
                                   (1, 32, 1024), (1, 33, 1024), (1, 2, 2048), (1, 2, 2049),
                                   (2, 16, 8193), (1, 2, 16384), (1, 2, 16385), (1, 9, 32768), (1, 2, 32769)])
def test_one_head(B, H, T):
    w, d = _inputs(B, H, H, T)
    c, mass = _select(w, d)
    _check(w, d, c, mass)
    _, shared = _select(w, d, mode=akvq.MODE_PSA_SHARED)
    assert ((shared.double() - mass.double()).abs() <= 8e-5 * mass.double() + 2e-12).all()


# several heads per KV head: rows whose stride is not a multiple of four, 256 keys and one more, as many workgroups as are
# resident at once and one head more, two to eight heads
@pytest.mark.parametrize("B,Hq,Hkv,T", [(1, 2, 1, 64), (3, 28, 4, 255), (40, 28, 4, 256), (1, 8, 1, 256), (65, 8, 1, 256), (18, 28, 4, 257), (19, 27, 9, 257),
                                        (128, 4, 2, 511), (129, 4, 2, 512), (1, 12, 2, 513), (8, 32, 8, 767), (9, 29, 29, 768), (9, 32, 8, 768),
                                        (1, 7, 1, 769), (2, 64, 8, 1025), (8, 16, 8, 2047), (8, 16, 8, 2049), (1, 8, 2, 32767), (1, 8, 1, 32768), (1, 9, 1, 512)])
def test_several_heads(B, Hq, Hkv, T):
    w, d = _inputs(B, Hq, Hkv, T)
    c, mass = _select(w, d)
    _check(w, d, c, mass)


@pytest.mark.parametrize("B,Hq,Hkv,T", [(1, 4, 4, 3000), (1, 28, 4, 400), (1, 12, 2, 1200), (17, 32, 32, 700)])
def test_smaller_workspaces_take_two_passes(B, Hq, Hkv, T):
    """What held the statistics of 2048-key chunks before still does; a byte less than the one pass needs takes two (or, up to
    768 keys with one head per KV head, the launch of a workgroup per head)."""
    w, d = _inputs(B, Hq, Hkv, T)
    full, up = akvq.lib().akvq_select_workspace_bytes(B, Hq, Hkv, T, 64), lambda n: (n + 255) // 256 * 256
    rest = up(B * Hkv * T * 4) + up(B * T * 4)
    once = up(B * Hq * -(-T // (512 if T > 768 or Hq == Hkv else T)) * 64 * 8) + rest + (up(B * Hq * -(-T // 4) * 16) if Hq > Hkv else 0)
    for nbytes in (full, once, once - 1, up(B * Hq * -(-T // 2048) * 64 * 8) + rest):
        c, mass = _select(w, d, nbytes=nbytes)
        _check(w, d, c, mass)


# a last chunk of one key, two batches of words, several rounds of heads, several heads per KV head
@pytest.mark.parametrize("B,Hq,Hkv,T", [(11, 2, 2, 1025), (1, 2, 2, 16800), (20, 32, 32, 900), (2, 12, 2, 1300)])
def test_missing_chunks_are_scored_by_who_waits(B, Hq, Hkv, T):
    """The same kernels built to look for a missing word once: a workgroup that does not find its siblings' statistics scores
    their chunks itself, to the same bits."""
    lib = C.CDLL(NOWAIT)
    w, d = _inputs(B, Hq, Hkv, T)
    c, mass = _select(w, d)
    c2, mass2 = _select(w, d, lib=lib)
    assert torch.equal(mass, mass2) and torch.equal(c.sal_idx, c2.sal_idx)


def test_replays_of_a_captured_selection():
    """New keys under the same graph, with eager work between the replays: the words of the replay before are cleared."""
    w, d = _inputs(2, 4, 4, 2500)
    c = akvq.Cache(w.B, w.Hkv, 128, 2560, 64, fill=0)
    mass = torch.zeros(w.B, w.Hkv, w.T, device="cuda")
    run = lambda: akvq.select_salient(c, akvq.MODE_PSA, q_tail=d["q_tail"], k=d["k"], top_k=8, sm_scale=w.sm_scale, mass_out=mass)  # noqa: E731
    run()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run()
    for seed in (1, 2, 3):
        _, other = _inputs(2, 4, 4, 2500, seed=seed)
        d["k"].copy_(other["k"])
        d["q_tail"].copy_(other["q_tail"])
        mass.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        got, idx = mass.clone(), c.sal_idx.clone()
        run()
        torch.cuda.synchronize()
        assert torch.equal(got, mass) and torch.equal(idx, c.sal_idx)


def test_beside_other_work():
    """Two selections of more workgroups than are resident, and a decode call, on three streams at once: the bits of each alone."""
    parts = [(w, d, akvq.Cache(w.B, w.Hkv, 128, (w.T + 63) // 64 * 64, 64, fill=0), torch.zeros(w.B, w.Hkv, w.T, device="cuda"))
             for w, d in (_inputs(12, 16, 16, 4500, seed=1), _inputs(3, 24, 24, 17000, seed=2))]
    w, d = _inputs(8, 16, 16, 2000, seed=3)
    c = akvq.Cache(w.B, w.Hkv, 128, 2048, 64, fill=0)
    akvq.quantize_append(c, d["k"], d["v"], 0.8)
    q = d["q_tail"][:, :, -1].contiguous()

    def select(i):
        w, d, c, mass = parts[i]
        akvq.select_salient(c, akvq.MODE_PSA, q_tail=d["q_tail"], k=d["k"], top_k=8, sm_scale=w.sm_scale, mass_out=mass)
        return mass, c.sal_idx

    calls = [lambda: select(0), lambda: select(1), lambda: akvq.decode_attention(c, q, w.sm_scale)]
    alone = []
    for call in calls:
        alone.append([t.clone() for t in call()])
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in calls]
    for _ in range(3):
        for _, _, cache, mass in parts:
            mass.fill_(float("nan"))
            cache.sal_idx.fill_(-1)
        torch.cuda.synchronize()
        got = []
        for stream, call in zip(streams, calls):
            with torch.cuda.stream(stream):
                got.append([t.clone() for t in call()])
        torch.cuda.synchronize()
        for one, other in zip(alone, got):
            assert all(torch.equal(x[..., :8] if x.dtype == torch.int32 else x, y[..., :8] if y.dtype == torch.int32 else y) for x, y in zip(one, other))
