"""The C-ABI library loads and exports every entry point include/akvq.h declares; host-only helpers behave.
No kernel is launched here (runs without a GPU)."""
import ctypes as C
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def L():
    from paper_2501_15021_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2501_15021_amd import build
        build.build()
    return binding.lib()


def test_every_declared_symbol_is_exported(L):
    from paper_2501_15021_amd import binding
    header = open(os.path.join(ROOT, "include", "akvq.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(akvq_[a-z_]+)\s*\(", header))
    assert declared == set(binding.EXPORTS)
    for name in declared:
        assert getattr(L, name) is not None


def test_host_helpers(L):
    from paper_2501_15021_amd.binding import akvq_cache
    assert L.akvq_version() >= 100
    assert L.akvq_strerror(0) == b"ok" and L.akvq_strerror(-3) == b"capacity exceeded"
    sizes = (C.c_size_t * 8)()
    shape = akvq_cache(2, 4, 128, 128, 64, 0)
    assert L.akvq_cache_bytes(C.byref(shape), sizes) == 0
    bh = 8
    assert list(sizes) == [bh * 4 * 1024, bh * 4 * 1024, bh * 128 * 4, bh * 128 * 4, bh * 64 * 256, bh * 64 * 256,
                           bh * 64 * 4, 32]
    shape64 = akvq_cache(2, 4, 64, 128, 64, 0)
    assert L.akvq_cache_bytes(C.byref(shape64), sizes) == 0 and sizes[2] == bh * 128 * 8
    for bad, code in ((akvq_cache(2, 4, 32, 128, 64, 0), -2), (akvq_cache(2, 4, 128, 100, 64, 0), -1),
                      (akvq_cache(0, 4, 128, 128, 64, 0), -1), (akvq_cache(2, 4, 128, 128, 64, 129), -3)):
        assert L.akvq_cache_bytes(C.byref(bad), sizes) == code
    assert L.akvq_decode_workspace_bytes(2, 8, 4) >= 2 * 8 * 4 * 132 * 4
    assert L.akvq_decode_workspace_bytes(0, 8, 4) == 0
    assert L.akvq_select_workspace_bytes(1, 32, 32, 640, 64) >= 32 * 1 * 64 * 2 * 4 + 32 * 640 * 4  # row statistics + masses
    for args in ((1, 32, 640), (16, 32, 4096), (64, 32, 8192), (32, 4, 32768), (1, 1, 1)):
        n = L.akvq_decode_default_splits(*args)
        assert 1 <= n <= 64 and n <= max(1, (args[2] + 63) // 64)


def test_decode_split_partition(L):
    """The KV-split partition the decode kernels use (the library exports the very function they call): the runs are
    disjoint, ordered and cover every tile; the split the fused decode step appends in is the one whose run holds the
    last tile -- also when trailing splits are empty (n_tiles < n_split, 5 tiles in 4 splits, ...), so the new row is
    written and read by the same workgroup."""
    b, e = C.c_int(), C.c_int()
    for n_tiles in list(range(0, 140)) + [289, 545, 1024, 1033]:
        for n_split in list(range(1, 70)) + [1024]:
            nxt, owner_seen = 0, None
            owner = None
            for s in range(n_split):
                owner = L.akvq_decode_split_range(n_tiles, n_split, s, C.byref(b), C.byref(e))
                assert 0 <= owner < n_split
                assert b.value == min(nxt, n_tiles) and b.value <= e.value <= n_tiles
                nxt = e.value
                if b.value <= n_tiles - 1 < e.value:
                    owner_seen = s
            assert nxt == n_tiles
            assert owner == (owner_seen if n_tiles else 0), (n_tiles, n_split)
    # the default split count at shapes where the last split is empty: the owner is not the last split
    for B, Hkv, T, rows in ((1, 28, 18433, 64), (2, 4, 34817, 32)):
        ns = L.akvq_decode_default_splits(B, Hkv, T)
        n_tiles = (T + rows - 1) // rows
        owner = L.akvq_decode_split_range(n_tiles, ns, 0, C.byref(b), C.byref(e))
        L.akvq_decode_split_range(n_tiles, ns, owner, C.byref(b), C.byref(e))
        assert b.value <= n_tiles - 1 < e.value
    assert L.akvq_decode_split_range(4, 0, 0, C.byref(b), C.byref(e)) == -1
    assert L.akvq_decode_split_range(4, 2, 2, C.byref(b), C.byref(e)) == -1
    assert L.akvq_decode_split_range(4, 2, 0, None, C.byref(e)) == -1


@pytest.mark.parametrize("Hq,Hkv", [(32, 32), (28, 4), (4, 4), (8, 1), (64, 8), (9, 1)])
@pytest.mark.parametrize("W", [16, 64])
def test_select_workspace_of_the_largest_call_serves_all(L, Hq, Hkv, W):
    """The size never shrinks when the batch or the prompt grows, and holds the statistics of at least one chunk per 2048
    keys beside the masses."""
    Ts = sorted({W, 640, *range(W, 70000, 997), *(2 ** n + d for n in range(7, 17) for d in (-1, 0, 1, 17))})
    Bs = [1, 2, 3, 4, 5, 7, 8, 9, 16, 17, 31, 32, 33, 64, 65, 128, 200]
    up = lambda n: (n + 255) // 256 * 256  # noqa: E731
    below = [0] * len(Ts)
    for B in Bs:
        sizes = [L.akvq_select_workspace_bytes(B, Hq, Hkv, T, W) for T in Ts]
        assert all(a <= b for a, b in zip(sizes, sizes[1:])), B
        assert all(a <= b for a, b in zip(below, sizes)), B
        for T, n in zip(Ts, sizes):
            assert n >= up(B * Hq * ((T + 2047) // 2048) * W * 8) + up(B * Hkv * T * 4) + up(B * T * 4)
        below = sizes


def test_argument_errors_launch_nothing(L):
    """Null pointers are rejected on the host before any launch (safe without a GPU)."""
    from paper_2501_15021_amd.binding import akvq_cache
    c = akvq_cache(1, 1, 128, 64, 64, 0)  # all device pointers null
    assert L.akvq_quantize_append(C.byref(c), None, None, 1, 0.8, 0, None) == -1
    assert L.akvq_decode_attention(C.byref(c), None, 1, 0.1, None, None, 1, None, 0, 0, None) == -1
    assert L.akvq_select_salient(C.byref(c), 0, None, None, 1, None, 64, 0, 0, 0.0, None, None, 0, None) == -1


def test_every_error_code_of_every_entry_point(L):
    """Each documented rejection, reached with well-formed fake device addresses: all of these return on the host before
    anything is launched or dereferenced, so they are safe without a GPU."""
    from paper_2501_15021_amd.binding import akvq_cache, akvq_window
    P = 0x7F0000001000                      # 16-byte aligned, never dereferenced
    INVALID, UNSUPPORTED, CAPACITY, WORKSPACE = -1, -2, -3, -4

    def cache(B=2, Hkv=2, G=128, T_cap=128, S_cap=64, T_len=0, **ptr):
        c = akvq_cache(B, Hkv, G, T_cap, S_cap, T_len, P, P, P, P, P, P, P, P)
        for k, v in ptr.items():
            setattr(c, k, v)
        return c

    big = 1 << 30
    # ---- write path
    q = L.akvq_quantize_append
    assert q(C.byref(cache(T_len=120)), P, P, 9, 0.8, 0, None) == CAPACITY
    assert q(C.byref(cache()), P, P, 0, 0.8, 0, None) == INVALID                 # no rows
    assert q(C.byref(cache()), P + 2, P, 4, 0.8, 0, None) == INVALID             # misaligned input
    assert q(C.byref(cache()), P, P, 4, 0.0, 0, None) == INVALID                 # clip outside (0, 1]
    assert q(C.byref(cache()), P, P, 4, 1.5, 0, None) == INVALID
    assert q(C.byref(cache(G=32)), P, P, 4, 0.8, 0, None) == UNSUPPORTED
    assert q(C.byref(cache(k_codes=None)), P, P, 4, 0.8, 0, None) == INVALID
    assert q(C.byref(cache(B=2048, Hkv=32)), P, P, 4, 0.8, 0, None) == UNSUPPORTED   # 65536 units: beyond the grid limit
    assert q(C.byref(cache(B=2047, Hkv=32, T_len=126)), P, P, 4, 0.8, 0, None) == CAPACITY   # 65504 units pass that check
    qt = L.akvq_quantize_append_tiered
    win = akvq_window(P, P, 96)                                                  # not a multiple of 64
    assert qt(C.byref(cache()), P, P, 4, None, None, 4, 0.8, 1.0, None, C.byref(win), 0, None) == INVALID
    win = akvq_window(None, P, 64)
    assert qt(C.byref(cache()), P, P, 4, None, None, 4, 0.8, 1.0, None, C.byref(win), 0, None) == INVALID
    assert qt(C.byref(cache()), P, P, 4, None, None, 4, 0.8, 1.5, None, None, 0, None) == INVALID   # 4-bit clip
    assert qt(C.byref(cache(T_len=100)), P, P, 4, P, P, 40, 0.8, 1.0, P, None, 0, None) == CAPACITY
    # ---- read path
    d = L.akvq_decode_attention
    assert d(C.byref(cache(T_len=0)), P, 2, 0.1, P, None, 1, P, big, 0, None) == INVALID            # empty cache
    assert d(C.byref(cache(T_len=5)), P, 3, 0.1, P, None, 1, P, big, 0, None) == INVALID            # Hq % Hkv
    assert d(C.byref(cache(T_len=5)), P, 18, 0.1, P, None, 1, P, big, 0, None) == UNSUPPORTED       # 9 heads per KV head
    assert d(C.byref(cache(T_len=5)), P, 2, 0.1, P, None, 2000, P, big, 0, None) == INVALID         # too many splits
    assert d(C.byref(cache(T_len=5)), P, 2, 0.1, P, None, 4, P, 64, 0, None) == WORKSPACE
    assert d(C.byref(cache(T_len=5)), P, 2, 0.1, P, None, 4, None, big, 0, None) == INVALID
    assert d(C.byref(cache(T_len=5)), P, 2, 0.1, P, P + 4, 1, P, big, 0, None) == INVALID           # misaligned lse
    assert d(C.byref(cache(B=16384, Hkv=4, T_len=5)), P, 4, 0.1, P, None, 1, P, 1 << 40, 0, None) == UNSUPPORTED   # grid limit
    dt = L.akvq_decode_attention_tiered
    assert dt(C.byref(cache(T_len=5)), P + 4, None, P, 2, 0.1, P, None, 1, P, big, 0, None) == INVALID
    win = akvq_window(P, P, 0)
    assert dt(C.byref(cache(T_len=5)), None, C.byref(win), P, 2, 0.1, P, None, 1, P, big, 0, None) == INVALID
    # ---- selection
    s = L.akvq_select_salient
    assert s(C.byref(cache()), 0, None, None, 2, None, 64, 0, 0, 0.0, None, None, 0, None) == INVALID      # no mask
    assert s(C.byref(cache()), 7, P, P, 2, P, 64, 16, 4, 0.1, None, P, big, None) == INVALID               # unknown mode
    assert s(C.byref(cache()), 1, None, P, 2, P, 200, 16, 4, 0.1, None, P, big, None) == INVALID           # T > T_cap
    assert s(C.byref(cache()), 1, None, P, 2, P, 64, 24, 4, 0.1, None, P, big, None) == UNSUPPORTED        # W % 16
    assert s(C.byref(cache()), 1, None, P, 2, P, 128, 128, 4, 0.1, None, P, big, None) == UNSUPPORTED      # W > 64
    assert s(C.byref(cache()), 1, None, P, 2, P, 64, 16, 65, 0.1, None, P, big, None) == CAPACITY
    assert s(C.byref(cache()), 1, None, P, 2, P, 64, 16, 4, 0.1, None, P, 16, None) == WORKSPACE
    assert s(C.byref(cache()), 1, None, P, 2, P, 8, 16, 4, 0.1, None, P, big, None) == INVALID             # W > T
    assert s(C.byref(cache(B=8192, Hkv=1)), 1, None, P, 8, P, 64, 16, 4, 0.1, None, P, 1 << 40, None) == UNSUPPORTED  # B*Hq
    m = L.akvq_select_massive
    assert m(C.byref(cache()), P, 64, 1000, 4, 0.0, None, P, big, None) == UNSUPPORTED                     # d_model % 512
    assert m(C.byref(cache()), P, 64, 1024, 65, 0.0, None, P, big, None) == CAPACITY
    assert m(C.byref(cache()), P, 64, 1024, 4, -1.0, None, P, big, None) == INVALID
    assert m(C.byref(cache()), P, 64, 1024, 4, float("nan"), None, P, big, None) == INVALID
    assert m(C.byref(cache()), P, 64, 1024, 4, 0.0, None, P, 16, None) == WORKSPACE
    assert m(C.byref(cache()), P, 64, 1024, 4, 0.0, None, None, 0, None) == INVALID
    assert m(C.byref(cache()), P, 300, 1024, 4, 0.0, None, P, big, None) == INVALID                        # T > T_cap
    # ---- fused rotary position embedding
    from paper_2501_15021_amd.binding import akvq_rope
    qr, dr = L.akvq_quantize_append_rope, L.akvq_decode_attention_rope
    ok, odd, nul = akvq_rope(P, P, 0), akvq_rope(P, P, 12), akvq_rope(P, None, 0)
    assert qr(C.byref(cache()), P, P, 4, None, None, 4, 0.8, 1.0, None, None, C.byref(ok), 4, None) == INVALID   # K pre-rotated
    assert qr(C.byref(cache()), P, P, 4, None, None, 4, 0.8, 1.0, None, None, C.byref(odd), 0, None) == INVALID  # stride % 8
    assert qr(C.byref(cache()), P, P, 4, None, None, 4, 0.8, 1.0, None, None, C.byref(nul), 0, None) == INVALID
    assert qr(C.byref(cache(T_len=126)), P, P, 4, None, None, 4, 0.8, 1.0, None, None, C.byref(ok), 0, None) == CAPACITY
    assert dr(C.byref(cache(T_len=5)), None, None, P, C.byref(ok), 2, 0.1, P, None, 1, P, big, 8, None) == INVALID  # q pre-rotated
    assert dr(C.byref(cache(T_len=5)), None, None, P, C.byref(nul), 2, 0.1, P, None, 1, P, big, 0, None) == INVALID
    assert dr(C.byref(cache(T_len=5)), None, None, P, C.byref(ok), 2, 0.1, P, None, 4, P, 64, 0, None) == WORKSPACE
    # ---- fused decode step
    ds = L.akvq_decode_step
    assert ds(C.byref(cache(T_len=128)), None, None, P, P, P, None, 2, 0.8, 0.1, P, None, 1, P, big, 0, None) == CAPACITY
    assert ds(C.byref(cache(T_len=5)), None, None, None, P, P, None, 2, 0.8, 0.1, P, None, 1, P, big, 0, None) == INVALID
    assert ds(C.byref(cache(T_len=5)), None, None, P, P, P, None, 2, 1.5, 0.1, P, None, 1, P, big, 0, None) == INVALID
    assert ds(C.byref(cache(T_len=5)), None, None, P, P, P, None, 3, 0.8, 0.1, P, None, 1, P, big, 0, None) == INVALID
    assert ds(C.byref(cache(T_len=5)), None, None, P, P, P, None, 2, 0.8, 0.1, P, None, 4, P, 64, 0, None) == WORKSPACE
    assert ds(C.byref(cache(T_len=5)), None, None, P, P, P, C.byref(ok), 2, 0.8, 0.1, P, None, 1, P, big, 4, None) == INVALID
    # ---- offline fold
    f = L.akvq_fold_hadamard
    assert f(P, P, 4, 100, 1, None) == INVALID                                   # columns not in runs of 128
    assert f(P, P + 4096, 100, 4, 0, None) == INVALID                            # rows not in runs of 128
    assert f(P, P, 128, 4, 0, None) == INVALID                                   # row fold cannot run in place
    assert f(P, P, 4, 128, 2, None) == INVALID
    assert f(None, P, 4, 128, 1, None) == INVALID
    sr = L.akvq_stream_read
    assert sr(None, 64, P, 1, None) == INVALID and sr(P, 8, P, 1, None) == INVALID and sr(P, 40, P, 0, None) == INVALID
    assert sr(P + 4, 64, P, 0, None) == INVALID and sr(P, 64, None, 1, None) == INVALID
    for code in (0, -1, -2, -3, -4, -5):
        assert len(L.akvq_strerror(code)) > 0


@pytest.mark.parametrize("B,Hkv", [(1, 1), (1, 2), (3, 2), (1, 32), (1, 40), (2, 32), (3, 32), (4, 32), (32, 4), (16, 32), (64, 32)])
def test_default_splits(L, B, Hkv):
    """One workgroup per CU at most with up to 64 units, at least two 64-row tiles each, none below 1024 rows; a workspace
    sized for the longest context serves every shorter one."""
    units, last = B * Hkv, 1
    for T in [1, 640, 1023, 1024, 1025, 1100, 2048, 3001, 8000, 20011, 32767, 32768, 34821, 200000]:
        n = L.akvq_decode_default_splits(B, Hkv, T)
        assert 1 <= n <= 64 and last <= n
        if units <= 64:
            assert units * n <= 256 and n <= max(1, (T + 63) // 64 // 2) and (T >= 1024 or n == 1)
        if units >= 512:
            assert n == 1
        last = n
