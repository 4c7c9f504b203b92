"""Infinities, NaN and the largest numbers among the keys and tail rows, W = 64: a row whose sum is no number spoils the masses of the
keys it sees, as dividing by that sum does, and of no others; every scoring kernel, and the two passes that little workspace gets."""
import ctypes as C

import pytest
import torch

from paper_2501_15021_amd import binding as akvq
from paper_2501_15021_amd import synth

pytestmark = pytest.mark.gpu
NAN, INF = float("nan"), float("inf")


def _masses(q, k, scale):
    """[T] of one KV head in binary64: q [R, 64, 128], k [T, 128]; keys a row does not see get nothing from it."""
    T = k.shape[0]
    seen = torch.arange(T, device="cuda")[None, :] <= (T - 64 + torch.arange(64, device="cuda"))[:, None]
    s = torch.matmul(q.bfloat16().double(), k.bfloat16().double().t().contiguous()) * scale
    top = torch.where(seen & ~s.isnan(), s, torch.full_like(s, -INF)).amax(dim=-1, keepdim=True)
    e = torch.where(seen, torch.exp(s - top), torch.zeros_like(s))
    return torch.where(seen, e / e.sum(dim=-1, keepdim=True), torch.zeros_like(s)).sum(dim=(0, 1))


# what lies where: tensor, position (negative: from the end) or tail row, channel, value
FAULTS = [("k", 5, 3, NAN), ("k", 5, 3, -NAN), ("k", 70, 0, INF), ("k", 70, 0, -INF), ("k", -1, 9, NAN), ("k", -20, 9, INF), ("k", -64, 9, INF),
          ("q", 0, 7, NAN), ("q", 40, 7, NAN), ("q", 63, 7, INF), ("q", 17, 0, -INF), ("q", 63, slice(None), NAN), ("k", -30, slice(None), NAN), None]


# one head per KV head: one launch, several chunks (the hidden keys in one and in two of them), two batches of words; several heads: one
# launch and a sum, several chunks; chunks of 2048 keys
@pytest.mark.parametrize("Hq,Hkv,T,B", [(2, 2, 300, 14), (2, 2, 700, 14), (2, 2, 1500, 14), (2, 2, 1025, 14), (1, 1, 17000, 14), (8, 4, 250, 14), (14, 2, 500, 14),
                                        (4, 2, 1100, 14), (4, 1, 4200, 600)])
@pytest.mark.parametrize("least", [False, True])
def test_nonfinite(Hq, Hkv, T, B, least):
    w = synth.small("nonfinite", B=B, Hq=Hq, Hkv=Hkv, T=T, G=128, n_text_head=5, n_text_tail=3, top_k=8, W=64)
    gen = torch.Generator(device="cuda").manual_seed(T)
    d = {n: torch.randn(B, H, rows, 128, generator=gen, device="cuda").half() for n, H, rows in (("q", Hq, 64), ("k", Hkv, T))}
    R, units = Hq // Hkv, {}
    for b, fault in enumerate(FAULTS):
        units[b] = b % Hkv
        if fault is not None:
            name, at, channel, value = fault
            d[name][b, units[b] * (R if name == "q" else 1), at, channel] = value
    up = lambda n: (n + 255) // 256 * 256  # noqa: E731
    nbytes = (up(B * Hq * -(-T // 2048) * 64 * 8) + up(B * Hkv * T * 4) + up(B * T * 4) if least
              else akvq.lib().akvq_select_workspace_bytes(B, Hq, Hkv, T, 64))
    c = akvq.Cache(B, Hkv, 128, (T + 63) // 64 * 64, 64, fill=0)
    ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")
    mass = torch.zeros(B, Hkv, T, device="cuda")
    s = c.struct()
    assert akvq.lib().akvq_select_salient(C.byref(s), akvq.MODE_PSA, None, d["q"].data_ptr(), Hq, d["k"].data_ptr(), T, 64, 8, w.sm_scale,
                                          mass.data_ptr(), ws.data_ptr(), nbytes, torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    wrong = []
    for b, h in units.items():
        want = _masses(d["q"][b, h * R:(h + 1) * R], d["k"][b, h], w.sm_scale)
        got = mass[b, h].double()
        if not torch.equal(got.isnan(), want.isnan()):
            wrong.append((FAULTS[b], int(got.isnan().sum()), int(want.isnan().sum())))
        # the bar of the pivot score: 4e-5 of the element (32-bit sums and exponentials), 1e-12 absolute
        elif not ((got - want).abs() <= 4e-5 * want + 1e-12)[~want.isnan()].all():
            wrong.append((FAULTS[b], "values"))
    assert wrong == []
    # largest bit pattern first, equal ones from the lowest position
    bits = mass.view(torch.int32).long() & 0xFFFFFFFF
    order = torch.sort(bits, dim=-1, descending=True, stable=True).indices[..., :8].sort(-1).values
    assert torch.equal(c.sal_idx[..., :8].long(), order) and (c.counts() == 8).all()
