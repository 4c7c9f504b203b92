"""Exact top-k at its borders: rows around the eight keys a thread requests together (256 and 1024 threads per workgroup),
many keys within a rounding step of the candidate bound, ties, and more candidates than the short cut ranks.  Scores are
handed in through akvq_select_massive, whose score is the largest magnitude of a token's hidden state."""
import pytest
import torch

from paper_2501_15021_amd import binding as akvq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,Hkv", [(7, 1), (255, 1), (2047, 2), (2048, 1), (2049, 1), (8191, 1), (8192, 1), (8193, 2), (12345, 1)])
@pytest.mark.parametrize("spread", ["random", "steps", "ties", "equal"])
def test_topk_of_given_scores(T, Hkv, spread):
    g = torch.Generator().manual_seed(T * 7 + len(spread))
    if spread == "random":
        score = torch.rand(T, generator=g).half() * 3
    elif spread == "steps":    # neighbouring binary16 numbers: up to four of them share the bound's sixteen bits
        score = (torch.randperm(T, generator=g) % 600 + 0x3C00).to(torch.int16).view(torch.float16)
    elif spread == "ties":
        score = torch.randint(1, 40, (T,), generator=g).half()
    else:                      # every key reaches the bound: the radix passes take over
        score = torch.full((T,), 1.5, dtype=torch.float16)
    hidden = torch.zeros(1, T, 512, dtype=torch.float16)
    hidden[0, torch.arange(T), torch.randint(0, 512, (T,), generator=g)] = score
    order = torch.sort(score.float(), descending=True, stable=True).indices
    c = akvq.Cache(1, Hkv, 128, (T + 63) // 64 * 64, 256, fill=0)
    hidden = hidden.cuda()
    for k in (1, 8, 64, 128, 200):
        akvq.select_massive(c, hidden, k)
        n = min(k, int((score > 0).sum()))
        assert (c.counts().cpu() == n).all()
        want = order[:n].sort().values.int()
        assert (c.sal_idx[0, :, :n].cpu() == want[None]).all(), (k, spread)


@pytest.mark.parametrize("T,Hkv", [(640, 4), (8191, 2), (9000, 2), (20000, 1)])
@pytest.mark.parametrize("gain", [0.0, 0.001, 0.003, 0.01, 0.03])
def test_topk_of_near_flat_masses(T, Hkv, gain):
    """Masses of nearly uniform attention: from all of the 256 maxima within the bound's sixteen bits to a part of them, so
    that the bound is searched to its last bit or not.  Sets against the stable order of the call's own masses."""
    g = torch.Generator(device="cuda").manual_seed(T)
    k = torch.randn(1, Hkv, T, 128, generator=g, device="cuda").half()
    q = (torch.randn(1, Hkv, 64, 128, generator=g, device="cuda") * gain).half()
    c = akvq.Cache(1, Hkv, 128, (T + 63) // 64 * 64, 256, fill=0)
    mass = torch.empty(1, Hkv, T, device="cuda")
    for top_k in (1, 8, 64, 128):
        akvq.select_salient(c, akvq.MODE_PSA, q_tail=q, k=k, top_k=top_k, sm_scale=128 ** -0.5, mass_out=mass)
        order = torch.sort(mass, dim=-1, descending=True, stable=True).indices[..., :top_k].sort(-1).values
        assert torch.equal(c.sal_idx[..., :top_k].long(), order), top_k
        assert (c.counts() == top_k).all()
