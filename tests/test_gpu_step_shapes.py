"""Fused decode steps at the borders of the decode kernels' launch shapes, against the oracle: four wavefronts per
workgroup (more than 256 workgroups) with the appended row in a wavefront's first, second, third and fourth tile (asked
for before or behind the append), up to and beyond 512 workgroups, and eight wavefronts (at most 256 workgroups), each
with and without a recent window and 4-bit row pairs."""
import numpy as np
import pytest
import torch

from paper_2501_15021_amd import binding as akvq
from paper_2501_15021_amd import synth

pytestmark = pytest.mark.gpu
ATTN_TOL = 2e-3
CLIP, SCALE = 0.8, 128 ** -0.5


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def _rows_plan(n_rows, tiers, B):
    """(number of source tokens, row plan or None) of a cache with n_rows rows (n_rows even where tiers are asked for)."""
    if not tiers:
        return n_rows, None
    T = n_rows
    while True:
        is_text = np.zeros((1, T), dtype=np.uint8)
        is_text[0, ::5] = 1
        src, tier, _ = synth.tiered_rows(is_text)
        if src.shape[1] <= n_rows:
            return T, (src.repeat(B, axis=0), tier.repeat(B, axis=0))
        T -= 1


def _steps(orc, B, Hkv, R, G, tiles, n_split, window, tiers, n_steps=2, slots=64):
    tile = 64 if R == 1 else 32
    # all steps append to the last of `tiles` tiles of every split's run
    T0, plan = _rows_plan((tiles * n_split - 1) * tile + tile // 2, tiers, B)
    rows0 = T0 if plan is None else plan[0].shape[1]
    assert rows0 // tile == (rows0 + n_steps - 1) // tile == tiles * n_split - 1
    t_cap = (rows0 + n_steps + 63) // 64 * 64
    rng = np.random.default_rng(B * 1000 + tiles * 10 + R)
    k, v = (rng.standard_normal((B, Hkv, T0 + n_steps, 128)).astype(np.float16) for _ in range(2))
    oc = orc.OracleCache(B, Hkv, G, t_cap, slots, fill=0)
    step, apart = (akvq.Cache(B, Hkv, G, t_cap, slots, fill=0) for _ in range(2))
    listed = [3, rows0 - 40, rows0 + 1] if plan is None else [rows0 + 1]  # one of the new rows is salient
    if slots > 64:
        listed = list(range(1, 2 * min(slots - 20, rows0 // 2 - 20), 2)) + listed[-1:]
    oc.sal_idx[:, :, :len(listed)] = listed
    oc.sal_cnt[:] = len(listed)
    for c in (step, apart):
        c.sal_idx.copy_(_dev(oc.sal_idx))
        c.counts().copy_(_dev(oc.sal_cnt))
    for c in (oc, step, apart):
        if window:
            c.enable_window(window)
    first = np.ascontiguousarray(k[:, :, :T0]), np.ascontiguousarray(v[:, :, :T0])
    rows = (None, None) if plan is None else plan
    oc.quantize_append_tiered(*first, *rows, CLIP, 1.0)
    for c in (step, apart):
        akvq.quantize_append_tiered(c, *map(_dev, first), *(None if r is None else _dev(r) for r in rows), CLIP, 1.0)
    for t in range(T0, T0 + n_steps):
        # a row whose absence would show in the output
        k1, v1 = k[:, :, t:t + 1] * np.float16(3), v[:, :, t:t + 1] * np.float16(50)
        q = (rng.standard_normal((B, Hkv, R, 128)) + np.sign(k1.astype(np.float64))).astype(np.float16).reshape(B, Hkv * R, 128)
        oc.quantize_append_tiered(k1, v1, None, None, CLIP, 1.0)
        ref, lse_ref = oc.decode(q, SCALE)
        out, lse = akvq.decode_step(step, _dev(k1), _dev(v1), _dev(q), CLIP, SCALE, n_split=n_split)
        akvq.quantize_append_tiered(apart, _dev(k1), _dev(v1), None, None, CLIP, 1.0)
        out2, lse2 = akvq.decode_attention(apart, _dev(q), SCALE, n_split=n_split)
        names = ("k_codes", "v_codes", "k_meta", "v_meta", "k_sal", "v_sal") + (("k_win", "v_win") if window else ())
        for n in names:
            assert torch.equal(getattr(step, n), getattr(apart, n)), (t, n)
        T = oc.T_len
        assert np.array_equal(step.k_meta.cpu().numpy().view(np.uint32)[:, :, :T], oc.k_meta[:, :, :T]), t
        assert np.array_equal(step.v_codes.cpu().numpy().view(np.uint32)[:, :, :T // 32], oc.v_codes[:, :, :T // 32]), t
        if n_split == 1:
            assert torch.equal(out, out2) and torch.equal(lse, lse2), f"fused vs separate calls, row {t}"
        rel = np.abs(out.cpu().numpy() - ref).max(-1) / np.maximum(np.abs(ref).max(-1), 1e-6)
        assert rel.max() <= ATTN_TOL, f"row {t}: {rel.max():.3e}"
        assert np.abs(lse.cpu().numpy() - lse_ref).max() <= 2e-3


@pytest.mark.parametrize("R,G", [(1, 128), (1, 64), (7, 64), (4, 128)])
@pytest.mark.parametrize("tiles", [4, 5, 8, 9, 13])
@pytest.mark.parametrize("window,tiers", [(0, False), (64, True)])
def test_four_wavefronts(orc, R, G, tiles, window, tiers):
    _steps(orc, 65, 4, R, G, tiles, 1, window, tiers)


@pytest.mark.parametrize("R,G", [(1, 64), (6, 64), (8, 128)])
@pytest.mark.parametrize("B", [64, 65])
def test_beyond_two_workgroups_per_cu(orc, R, G, B):  # 512 and 520 workgroups
    _steps(orc, B, 8, R, G, 6, 1, 0, True, n_steps=1)


@pytest.mark.parametrize("R,G", [(1, 128), (1, 64), (7, 64), (4, 128)])
@pytest.mark.parametrize("tiles,n_split", [(8, 1), (17, 1), (26, 1), (9, 2)])
@pytest.mark.parametrize("window,tiers", [(0, False), (64, False), (0, True), (128, True)])
def test_eight_wavefronts(orc, R, G, tiles, n_split, window, tiers):
    _steps(orc, 2, 3, R, G, tiles, n_split, window, tiers)


# up to four tiles a split, but a step with more 16-bit rows than four wavefronts have units for: eight all the same
@pytest.mark.parametrize("R,G,window,slots", [(7, 64, 512, 64), (4, 128, 128, 64), (6, 64, 0, 192), (1, 128, 0, 256), (1, 64, 512, 192)])
@pytest.mark.parametrize("tiles,n_split", [(2, 8), (4, 3)])
@pytest.mark.parametrize("tiers", [False, True])
def test_eight_wavefronts_of_few_tiles(orc, R, G, window, slots, tiles, n_split, tiers):
    _steps(orc, 2, 3, R, G, tiles, n_split, window, tiers, slots=slots if not tiers else 64 if slots == 64 else 128)


# 16-bit rows two units at a time (more than one workgroup per CU and more units than wavefronts, or more than two per CU), with
# odd numbers of units, windows that are not full yet and long salient lists
@pytest.mark.parametrize("Hkv,window,slots,tiles", [(4, 128, 64, 5), (4, 512, 64, 3), (4, 192, 192, 7), (4, 0, 256, 8), (8, 64, 64, 2), (8, 0, 64, 2),
                                                    (8, 512, 64, 1), (8, 128, 128, 5)])
@pytest.mark.parametrize("G,tiers", [(128, False), (64, False), (128, True), (64, True)])
def test_pairs_of_row_units(orc, Hkv, window, slots, tiles, G, tiers):
    _steps(orc, 65, Hkv, 1, G, tiles, 1, window, tiers, slots=slots if not tiers else min(slots, 128))


@pytest.mark.parametrize("window,slots,tiles", [(256, 64, 4), (256, 64, 9), (512, 64, 12), (0, 320, 11), (192, 192, 3)])  # a workgroup per CU
@pytest.mark.parametrize("G,tiers", [(128, False), (64, True)])
def test_pairs_of_row_units_with_four_and_eight_wavefronts(orc, window, slots, tiles, G, tiers):
    _steps(orc, 64, 4, 1, G, tiles, 1, window, tiers, slots=slots if not tiers else min(slots, 128))
