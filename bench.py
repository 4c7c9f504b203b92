#!/usr/bin/env python3
"""Benchmark of the AKVQ-VL KV-cache hot path on one MI355X.

A step is one pass of the whole hot path over one batch of synthetic input, for every layer of the workload:
  akvq_select_salient (TSA layers: text mask; PSA layers: attention-column mass + top-k)
  -> akvq_quantize_append (rotate, 2-bit quantize, pack, bf16 overlay for salient rows; the whole prompt)
  -> akvq_decode_attention (one decode query per head over the packed cache).
Inputs are resident in HBM before the timed region.  Prints ONE JSON line.

  python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload cfg2]
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBPS = 8000.0  # MI355X HBM3E, published
ALU_PEAK_GLANEOPS = 256 * 64 * 2.4   # fp32 vector lane-operations per ns without packed fp32 (= 78.6 TFLOP/s as FMAs)
# HBM bytes per launch counted by rocprofv3 --pmc (FETCH_SIZE x 2.000 + WRITE_SIZE x 1.000 KiB, factors from a 1 GiB
# copy), mean over the 32 layers of cfg2; runs and raw figures in profiles/bench_cfg2_kernel_trace.md.  The counters
# cannot be read from inside this process, so the figures are stored with a hash of the kernel sources they were
# measured on and reported as roofline.traffic only while the sources still hash to that value (null otherwise, and
# for every other workload).
MEASURED_TRAFFIC = {"source_hash": "f476ed9244a9ea3c",
                    "cfg2": {"quantize": 1257826496, "select": 612216877, "decode": 174444134}}


def kernel_source_hash():
    import glob
    import hashlib
    h = hashlib.sha256()
    for path in sorted(glob.glob(os.path.join(ROOT, "paper_2501_15021_amd", "csrc", "*.h*"))):
        h.update(os.path.basename(path).encode())
        h.update(open(path, "rb").read())
    return h.hexdigest()[:16]


METRIC = "decode-attn KV tokens/s/GPU + achieved HBM GB/s (% peak); quantize GB/s"


def algorithmic_bytes(w, layer):
    """Bytes each call must move at least once (per layer)."""
    bh = w.B * w.Hkv
    per_row = 2 * (32 + 4 * (128 // w.G))                      # K+V codes and meta of one cached row
    n_sal = w.n_text if w.mode(layer) == "tsa" else w.top_k
    decode = bh * ((w.T - n_sal) * per_row + n_sal * 512)        # salient rows are read as bf16 instead
    quant_in = bh * w.T * 128 * 2 * 2                            # fp16 K and V
    quant_out = bh * (w.T * per_row + n_sal * 512)
    score = 0 if w.mode(layer) == "tsa" else bh * w.T * 128 * 2   # K once (some shapes are scored in two passes)
    return {"decode": decode, "quantize": quant_in + quant_out, "quantize_in": quant_in, "select": score}


def cpu_baseline(w, layer, data):
    """The oracle as it stands, on this machine's host cores, on one layer of the same workload."""
    import numpy as np
    from oracle import pyoracle as orc
    host = {k: data[k].cpu().numpy() for k in ("k", "v", "q", "q_tail", "is_text")}
    oc = orc.OracleCache(w.B, w.Hkv, w.G, (w.T + 63) // 64 * 64, w.s_cap(layer))
    t0 = time.perf_counter()
    if w.mode(layer) == "tsa":
        oc.select_tsa(host["is_text"])
    else:
        mass = oc.select_psa(host["q_tail"], host["k"], w.top_k, w.sm_scale, want_mass=True)
    t1 = time.perf_counter()
    oc.quantize_append(host["k"], host["v"], w.clip)
    t2 = time.perf_counter()
    oc.decode(host["q"], w.sm_scale)
    t3 = time.perf_counter()
    cores = int(os.environ.get("OMP_NUM_THREADS", os.cpu_count() or 1))
    oc.margins = orc.topk_margins(mass, w.top_k) if w.mode(layer) == "psa" else None   # after the timed part
    return {"value": w.B * w.T / (t3 - t0), "unit": "KV tokens/s", "cores": cores, "kind": "oracle",
            "sample": f"one {w.mode(layer).upper()} layer (layer {layer}) of {w.name}: B={w.B}, {w.Hkv} heads, T={w.T}",
            "seconds": {"select": round(t1 - t0, 3), "quantize": round(t2 - t1, 3), "decode": round(t3 - t2, 3)},
            "decode_kv_tokens_per_s": w.B * w.T / (t3 - t2)}, oc


def decode_alone(w, akvq, synth, torch, np, warmup=20, timed=100, n_split=0):
    """akvq_decode_attention alone on workload w (a pivot-salient layer), rotating through distinct caches that
    together exceed the last-level cache several times; HIP events on the launch stream around `timed` launches."""
    layer = 2 if w.tsa_layers else 0
    per_set = algorithmic_bytes(w, layer)["decode"]
    n_sets = max(2, int(np.ceil(1.2e9 / per_set)))
    t_cap = (w.T + 63) // 64 * 64
    sets = []
    for i in range(n_sets):
        d = synth.generate(w, layer=layer + 100 * i, device="cuda")
        cache = akvq.Cache(w.B, w.Hkv, w.G, t_cap, w.s_cap(layer))
        akvq.select_salient(cache, akvq.MODE_PSA, q_tail=d["q_tail"], k=d["k"], top_k=w.top_k, sm_scale=w.sm_scale)
        akvq.quantize_append(cache, d["k"], d["v"], w.clip)
        torch.cuda.synchronize()
        sets.append((d["q"], cache))
        del d
    out = torch.empty(w.B, w.Hq, 128, device="cuda")
    lse = torch.empty(w.B, w.Hq, device="cuda")
    for i in range(warmup):
        akvq.decode_attention(sets[i % n_sets][1], sets[i % n_sets][0], w.sm_scale, n_split=n_split, out=out, lse=lse)
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for i in range(timed):
        akvq.decode_attention(sets[i % n_sets][1], sets[i % n_sets][0], w.sm_scale, n_split=n_split, out=out, lse=lse)
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / timed
    gbps = per_set / (ms * 1e-3) / 1e9
    ns = n_split or akvq.lib().akvq_decode_default_splits(w.B, w.Hkv, w.T)
    return {"kernel": ("decode_mha_kernel" if w.Hq == w.Hkv else "decode_gqa_kernel") + (" + decode_combine_kernel" if ns > 1 else ""),
            "workload": f"{w.name}: B={w.B} x Hq={w.Hq}/Hkv={w.Hkv} x T={w.T}, G={w.G}, PSA top-{w.top_k}",
            "bound": "hbm", "achieved": round(gbps, 1), "peak": HBM_PEAK_GBPS, "unit": "GB/s",
            "frac": round(gbps / HBM_PEAK_GBPS, 4), "traffic": None, "avg_launch_ms": round(ms, 5),
            "algorithmic_bytes_per_launch": per_set, "launches_timed": timed, "warmup_launches": warmup,
            "buffer_sets": n_sets, "n_split": ns, "kv_tokens_per_s": w.B * w.T / (ms * 1e-3)}


def prefill_alone(w, akvq, synth, torch, np, warmup=3, timed=20):
    """akvq_select_salient (pivot selection) and akvq_quantize_append alone on one pivot-salient layer of workload w,
    two input sets alternating; HIP events around `timed` calls of each."""
    layer = 2 if w.tsa_layers else 0
    t_cap = (w.T + 63) // 64 * 64
    sets = []
    for i in range(2):
        d = synth.generate(w, layer=layer + 100 * i, device="cuda")
        sets.append((d["q_tail"], d["k"], d["v"], akvq.Cache(w.B, w.Hkv, w.G, t_cap, w.s_cap(layer))))
        del d

    def timed_ms(fn):
        for i in range(warmup):
            fn(sets[i % 2])
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for i in range(timed):
            fn(sets[i % 2])
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / timed

    def select(s):
        akvq.select_salient(s[3], akvq.MODE_PSA, q_tail=s[0], k=s[1], top_k=w.top_k, sm_scale=w.sm_scale)

    def quantize(s):
        s[3].T_len = 0
        akvq.quantize_append(s[3], s[1], s[2], w.clip)

    sel_ms, q_ms = timed_ms(select), timed_ms(quantize)
    b = algorithmic_bytes(w, layer)
    return {"workload": f"{w.name}: B={w.B} x Hq={w.Hq}/Hkv={w.Hkv} x T={w.T}, G={w.G}, PSA top-{w.top_k}",
            "select_ms": round(sel_ms, 4), "select_GBps": round(b["select"] / (sel_ms * 1e-3) / 1e9, 1),
            "quantize_ms": round(q_ms, 4), "quantize_GBps": round(b["quantize"] / (q_ms * 1e-3) / 1e9, 1),
            "quantize_frac_of_hbm_peak": round(b["quantize"] / (q_ms * 1e-3) / 1e9 / HBM_PEAK_GBPS, 4),
            "calls_timed": timed}


def stream_ceiling(akvq, torch, warmup=5, timed=40):
    """GB/s of the plain 128-bit streaming-read kernel over two 2 GiB buffers (alternating: no reuse in any cache),
    with the non-temporal load hint the decode kernels use and without it."""
    n = 1 << 31
    bufs = [torch.empty(n, dtype=torch.uint8, device="cuda").random_(0, 255) for _ in range(2)]
    sink = torch.zeros(4, dtype=torch.int32, device="cuda")
    res = {"kernel": "stream_read_kernel", "bytes_per_launch": n, "launches_timed": timed}
    for name, nt in (("non_temporal", True), ("plain", False)):
        for i in range(warmup):
            akvq.stream_read(bufs[i % 2], sink, nt)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for i in range(timed):
            akvq.stream_read(bufs[i % 2], sink, nt)
        e1.record()
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / timed
        res[name] = {"avg_launch_ms": round(ms, 4), "GBps": round(n / (ms * 1e-3) / 1e9, 1),
                     "frac_of_hbm_peak": round(n / (ms * 1e-3) / 1e9 / HBM_PEAK_GBPS, 4)}
    res["GBps"] = max(res["non_temporal"]["GBps"], res["plain"]["GBps"])
    return res


def oracle_bench(args, w, synth, torch, np):
    """The CPU oracle at the workload's full size (one layer), on all host threads: seconds per call, effective GB/s."""
    from oracle import pyoracle as orc
    layer = args.layer if args.layer >= 0 else (2 if w.tsa_layers else 0)
    d = synth.generate(w, layer=layer, device="cuda" if torch.cuda.is_available() else "cpu")
    host = {k: d[k].cpu().numpy() for k in ("k", "v", "q", "q_tail", "is_text")}
    del d
    oc = orc.OracleCache(w.B, w.Hkv, w.G, (w.T + 63) // 64 * 64, w.s_cap(layer))
    t0 = time.perf_counter()
    if w.mode(layer) == "tsa":
        oc.select_tsa(host["is_text"])
    else:
        oc.select_psa(host["q_tail"], host["k"], w.top_k, w.sm_scale)
    t1 = time.perf_counter()
    print(f"oracle {w.name}: select {t1 - t0:.2f} s", file=sys.stderr, flush=True)
    oc.quantize_append(host["k"], host["v"], w.clip)
    t2 = time.perf_counter()
    print(f"oracle {w.name}: quantize {t2 - t1:.2f} s", file=sys.stderr, flush=True)
    oc.decode(host["q"], w.sm_scale)
    t3 = time.perf_counter()
    ab = algorithmic_bytes(w, layer)
    cores = int(os.environ.get("OMP_NUM_THREADS", os.cpu_count() or 1))
    print(json.dumps({"metric": "CPU oracle at full size (one layer)", "workload": w.name, "layer_mode": w.mode(layer),
                      "cores": cores, "nproc": os.cpu_count(),
                      "seconds": {"select": round(t1 - t0, 3), "quantize": round(t2 - t1, 3), "decode": round(t3 - t2, 3)},
                      "effective_GBps": {"select": round(ab["select"] / max(t1 - t0, 1e-9) / 1e9, 3),
                                         "quantize": round(ab["quantize"] / (t2 - t1) / 1e9, 3),
                                         "decode": round(ab["decode"] / (t3 - t2) / 1e9, 3)},
                      "kv_tokens_per_s": {"decode": w.B * w.T / (t3 - t2), "whole_path": w.B * w.T / (t3 - t0)}}))


def phase_bench(args, w, akvq, synth, torch, np):
    """Time one call of the path on its own, rotating through distinct buffer sets larger than the last-level cache."""
    layer = 0 if not w.tsa_layers else 2          # a PSA layer when the workload has both kinds
    if w.mode(layer) == "tsa":
        layer = 0
    if args.layer >= 0:
        layer = args.layer                        # e.g. --layer 0 times a text-salient layer of cfg2
    per_set = algorithmic_bytes(w, layer)
    n_sets = args.sets or max(2, int(np.ceil(1.2e9 / max(per_set["decode"], 1))) if args.phase == "decode" else 2)
    t_cap = (w.T + 63) // 64 * 64
    sets = []
    for i in range(n_sets):
        d = synth.generate(w, layer=layer + 100 * i, device="cuda")
        cache = akvq.Cache(w.B, w.Hkv, w.G, t_cap, w.s_cap(layer))
        sets.append((d, cache))

    if args.window:
        for _, cache in sets:
            cache.enable_window(args.window)
    tiered = None
    if args.tiered:
        # Section III-C.1 tiers: text tokens (all but position 0, a planted pivot) 4-bit as row pairs, pivot tokens
        # 16-bit, the rest 2-bit.  The row plan depends on the prompt layout only, so it is built once on the host.
        mask = sets[0][0]["is_text"].cpu().numpy()
        row_src, row_tier, row_of = synth.tiered_rows(mask, [[0]] * w.B)
        n_rows = row_src.shape[1]
        t_cap = (n_rows + 63) // 64 * 64
        tiered = {"row_src": torch.from_numpy(row_src).cuda(), "row_tier": torch.from_numpy(row_tier).cuda(),
                  "row_of": torch.from_numpy(row_of).cuda().long(), "n_rows": n_rows,
                  "plain": torch.from_numpy(((mask == 0) | (np.arange(w.T)[None, :] == 0))).cuda()}
        sets = [(d, akvq.Cache(w.B, w.Hkv, w.G, t_cap, w.s_cap(layer))) for d, _ in sets]
        if args.window:
            for _, cache in sets:
                cache.enable_window(args.window)
        n_pairs = int((row_tier == 2).sum(axis=1).max())
        per_row = 2 * (32 + 4 * (128 // w.G))
        per_set = dict(per_set)
        per_set["decode"] = w.B * w.Hkv * ((n_rows - w.top_k) * per_row + w.top_k * 512)
        per_set["quantize"] = per_set["quantize_in"] + w.B * w.Hkv * (n_rows * per_row + w.top_k * 512)

    def to_rows(cache):
        """salient token positions -> cache rows, keeping only tokens stored as plain rows (ascending order kept)"""
        idx = cache.sal_idx.long().clamp_(min=0)
        cnt = cache.counts().clamp(max=cache.S_cap)
        b_ix = torch.arange(w.B, device=idx.device)[:, None, None].expand_as(idx)
        ok = (torch.arange(cache.S_cap, device=idx.device)[None, None, :] < cnt[:, :, None]) & tiered["plain"][b_ix, idx]
        rows = torch.where(ok, tiered["row_of"][b_ix, idx], torch.full_like(idx, 1 << 30))
        rows, _ = torch.sort(rows, dim=-1)
        cache.sal_idx.copy_(torch.where(rows < (1 << 30), rows, torch.full_like(rows, -1)).int())
        cache.counts().copy_(ok.sum(-1).int())

    rope = None
    if args.rope:  # K rows are taken as pre-RoPE and embedded inside the write path (timing only: same bytes)
        rope = tuple(torch.from_numpy(t).cuda() for t in synth.rope_tables(np.arange(w.T)))

    def append(d, cache):
        if tiered:
            akvq.quantize_append_tiered(cache, d["k"], d["v"], tiered["row_src"], tiered["row_tier"], w.clip, 1.0,
                                        rope=rope)
        elif args.window or rope:
            akvq.quantize_append_tiered(cache, d["k"], d["v"], None, None, w.clip, 1.0, rope=rope)
        else:
            akvq.quantize_append(cache, d["k"], d["v"], w.clip)

    def prepare(d, cache, upto):
        cache.T_len = 0
        if w.mode(layer) == "tsa":
            akvq.select_salient(cache, akvq.MODE_TSA, is_text=d["is_text"])
        else:
            akvq.select_salient(cache, akvq.MODE_PSA, q_tail=d["q_tail"], k=d["k"], top_k=w.top_k, sm_scale=w.sm_scale)
        if tiered:
            to_rows(cache)
        if upto == "select":
            return
        append(d, cache)

    def call(d, cache):
        if args.phase == "decode":
            akvq.decode_attention(cache, d["q"], w.sm_scale, n_split=args.n_split)
        elif args.phase == "quantize":
            cache.T_len = 0
            append(d, cache)
        else:
            prepare(d, cache, "select")

    for d, cache in sets:
        prepare(d, cache, "quantize" if args.phase == "decode" else "select")
    if args.phase == "decode":      # the inputs are no longer needed: keep HBM for the caches
        for d, _ in sets:
            d.pop("k"); d.pop("v")
    torch.cuda.synchronize()
    for i in range(args.warmup * n_sets):
        call(*sets[i % n_sets])
    torch.cuda.synchronize()
    n_calls = args.steps * n_sets
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for i in range(n_calls):
        call(*sets[i % n_sets])
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / n_calls
    nbytes = per_set[args.phase]
    if args.window:  # window rows are read (decode) / also written (quantize) as 16-bit instead of / besides their codes
        per_row = 2 * (32 + 4 * (128 // w.G))
        nbytes += w.B * w.Hkv * args.window * (512 - per_row if args.phase == "decode" else 512)
    gbps = nbytes / (ms * 1e-3) / 1e9
    out = {"metric": f"{args.phase} call alone" + (" (4-bit text tier as row pairs)" if tiered else ""),
           "cache_rows": tiered["n_rows"] if tiered else w.T, "recent_window": args.window, "fused_rope": bool(args.rope), "workload": w.name, "layer_mode": w.mode(layer), "ms_per_call": round(ms, 5),
           "kv_tokens_per_s": w.B * w.T / (ms * 1e-3), "n_sets": n_sets, "calls": n_calls,
           "n_split": args.n_split or akvq.lib().akvq_decode_default_splits(w.B, w.Hkv, w.T),
           "roofline": {"bound": "hbm", "achieved": round(gbps, 1), "peak": HBM_PEAK_GBPS, "unit": "GB/s",
                        "frac": round(gbps / HBM_PEAK_GBPS, 4), "traffic": None,
                        "algorithmic_bytes_per_launch": nbytes}}
    if args.phase == "quantize":
        out["input_GBps"] = round(per_set["quantize_in"] / (ms * 1e-3) / 1e9, 1)
    print(json.dumps(out))


def capacity_bench(args, w, akvq, synth, torch, np):
    """One-GPU analogue of the paper's capacity / throughput comparison (Section IV-D, Table IV): at a fixed HBM budget
    for the KV cache, the largest batch a 16-bit cache and the mixed 2-bit cache hold at this context length, and the
    decode-attention rate of each at its largest batch.  One layer's share of the budget is allocated and timed (all
    layers have the same shape); the 16-bit cache is this library's own format with every row in the 16-bit window."""
    import ctypes as C
    import dataclasses
    L, T = args.layers or w.n_layers, w.T
    t_cap = (T + 63) // 64 * 64
    layer = 2 if w.tsa_layers else 0                     # a pivot-token layer (all but two layers of cfg2)
    budget = args.budget_gb * 1e9 / L
    sizes = (C.c_size_t * 8)()
    shape = akvq.akvq_cache(1, w.Hkv, w.G, t_cap, w.s_cap(layer), 0)
    assert akvq.lib().akvq_cache_bytes(C.byref(shape), sizes) == 0
    bytes2 = sum(sizes)
    bytes16 = 2 * w.Hkv * t_cap * 256
    b16, b2 = int(budget // bytes16), int(budget // bytes2)
    chunk = min(8, b16)
    wc = dataclasses.replace(w, B=chunk)

    def build(B, sixteen):
        big = akvq.Cache(B, w.Hkv, w.G, t_cap, w.s_cap(layer))
        if sixteen:
            big.enable_window(t_cap)
        smalls = []
        for i in range(3):                               # three distinct chunks, dealt round-robin over the batch
            d = synth.generate(wc, layer=layer + 100 * i, device="cuda")
            c = akvq.Cache(chunk, w.Hkv, w.G, t_cap, w.s_cap(layer))
            if sixteen:
                c.enable_window(t_cap)
                akvq.quantize_append_tiered(c, d["k"], d["v"], None, None, w.clip, 1.0)
            else:
                akvq.select_salient(c, akvq.MODE_PSA, q_tail=d["q_tail"], k=d["k"], top_k=w.top_k, sm_scale=w.sm_scale)
                akvq.quantize_append(c, d["k"], d["v"], w.clip)
            smalls.append(c)
            del d
        names = ["k_codes", "v_codes", "k_meta", "v_meta", "k_sal", "v_sal", "sal_idx"] + (["k_win", "v_win"] if sixteen else [])
        for i, b0 in enumerate(range(0, B, chunk)):
            n = min(chunk, B - b0)
            src = smalls[i % 3]
            for name in names:
                getattr(big, name)[b0:b0 + n].copy_(getattr(src, name)[:n])
            big.counts()[b0:b0 + n].copy_(src.counts()[:n])
        big.T_len = T
        return big

    def time_decode(cache):
        g = torch.Generator(device="cuda").manual_seed(5)
        q = torch.randn(cache.B, w.Hq, 128, generator=g, device="cuda").half()
        for _ in range(args.warmup):
            akvq.decode_attention(cache, q, w.sm_scale)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(args.steps):
            akvq.decode_attention(cache, q, w.sm_scale)
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / args.steps

    res = {}
    for name, B, sixteen in (("16-bit cache, its largest batch", b16, True), ("2-bit cache, the same batch", b16, False),
                             ("2-bit cache, its largest batch", b2, False)):
        cache = build(B, sixteen)
        ms = time_decode(cache)
        per_row = 2 * (32 + 4 * (128 // w.G))
        nbytes = B * w.Hkv * (T * 512 if sixteen else (T - w.top_k) * per_row + w.top_k * 512)
        res[name] = {"batch": B, "cache_GB_all_layers": round(B * (bytes16 if sixteen else bytes2) * L / 1e9, 1),
                     "ms_per_layer": round(ms, 4), "decode_tokens_per_s_attention_only": round(B / (L * ms * 1e-3), 1),
                     "GBps": round(nbytes / (ms * 1e-3) / 1e9, 1)}
        del cache
        torch.cuda.empty_cache()
    r16, r2 = res["16-bit cache, its largest batch"], res["2-bit cache, its largest batch"]
    ideal16 = b16 / (L * (b16 * w.Hkv * T * 512) / (HBM_PEAK_GBPS * 1e9))
    print(json.dumps({"metric": "capacity and decode-attention rate at a fixed KV-cache budget", "workload": w.name,
                      "context": T, "layers": L, "budget_GB": args.budget_gb,
                      "bytes_per_sequence_per_layer": {"16-bit": bytes16, "2-bit mixed": bytes2},
                      "max_batch_ratio": round(b2 / b16, 3), **res,
                      "throughput_ratio_at_max_batch": round(r2["decode_tokens_per_s_attention_only"] /
                                                             r16["decode_tokens_per_s_attention_only"], 3),
                      "16-bit cache at the HBM peak (bound, not measured)": round(ideal16, 1),
                      "throughput_ratio_vs_that_bound": round(r2["decode_tokens_per_s_attention_only"] / ideal16, 3)}))


def decode_step_bench(args, w, akvq, synth, torch, np):
    """One generated token through the cache of every layer: per layer, append the new token's K and V (rotary
    embedding fused in) and run decode attention over the cache.  Launch-bound at small batch; --graph replays the
    whole step as one HIP graph (the library allocates nothing and records no memset, so it can be captured)."""
    L = args.layers or w.n_layers
    t_cap = (w.T + 64) // 64 * 64
    caches, qs, news = [], [], []
    rope_all = tuple(torch.from_numpy(t).cuda() for t in synth.rope_tables(np.arange(w.T)))
    rope_new = tuple(torch.from_numpy(t).cuda() for t in synth.rope_tables(np.array([w.T])))
    for layer in range(L):
        d = synth.generate(w, layer=layer, device="cuda")
        c = akvq.Cache(w.B, w.Hkv, w.G, t_cap, w.s_cap(layer))
        if w.mode(layer) == "tsa":
            akvq.select_salient(c, akvq.MODE_TSA, is_text=d["is_text"])
        else:
            akvq.select_salient(c, akvq.MODE_PSA, q_tail=d["q_tail"], k=d["k"], top_k=w.top_k, sm_scale=w.sm_scale)
        akvq.quantize_append_tiered(c, d["k"], d["v"], None, None, w.clip, 1.0, rope=rope_all)
        caches.append(c)
        qs.append(d["q"])
        news.append((d["k"][:, :, :1].contiguous(), d["v"][:, :, :1].contiguous()))
        del d
    out = torch.empty(w.B, w.Hq, 128, device="cuda")
    lse = torch.empty(w.B, w.Hq, device="cuda")

    def step():
        for c, q, (k1, v1) in zip(caches, qs, news):
            c.T_len = w.T
            if args.fused:   # akvq_decode_step: the append runs inside the decode launch
                akvq.decode_step(c, k1, v1, q, w.clip, w.sm_scale, out=out, lse=lse, rope=rope_new)
            else:
                akvq.quantize_append_tiered(c, k1, v1, None, None, w.clip, 1.0, rope=rope_new)
                akvq.decode_attention(c, q, w.sm_scale, out=out, lse=lse, rope=rope_new)

    for _ in range(max(args.warmup, 1)):
        step()
    torch.cuda.synchronize()
    run = step
    if args.graph:
        graph = torch.cuda.CUDAGraph()
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            with torch.cuda.graph(graph, stream=side):
                step()
        torch.cuda.synchronize()
        run = graph.replay
        run()
        torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(args.steps):
        run()
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / args.steps
    per_row = 2 * (32 + 4 * (128 // w.G))
    nbytes = sum(w.B * w.Hkv * ((w.T + 1 - min(w.s_cap(l), w.n_text if w.mode(l) == "tsa" else w.top_k)) * per_row
                                + (w.n_text if w.mode(l) == "tsa" else w.top_k) * 512) for l in range(L))
    print(json.dumps({"metric": "decode step over all layers (append one token + decode attention)",
                      "workload": w.name, "layers": L, "batch": w.B, "context": w.T + 1, "hip_graph": bool(args.graph), "fused_append": bool(args.fused),
                      "ms_per_step": round(ms, 4), "launches_per_step": (1 if args.fused else 2) * L,
                      "generated_tokens_per_s_attention_path": round(w.B / (ms * 1e-3), 1),
                      "cache_GBps": round(nbytes / (ms * 1e-3) / 1e9, 1),
                      "frac_of_hbm_peak": round(nbytes / (ms * 1e-3) / 1e9 / HBM_PEAK_GBPS, 4)}))


def ablation_bench(args, w, akvq, synth, torch, np):
    """Synthetic-data analogue of the paper's ablation (Section IV-C, Table III): error of the decode-attention output
    against exact attention over the unquantized K and V, with and without the rotation and the 16-bit salient tokens.
    The inputs are this build's synthetic ones (outlier channels in K, planted pivot rows), not the paper's benchmark."""
    import dataclasses
    w = dataclasses.replace(w, B=min(w.B, 4))
    layer = 2 if w.tsa_layers else 0
    d = synth.generate(w, layer=layer, device="cuda")
    t_cap = (w.T + 63) // 64 * 64
    r = w.Hq // w.Hkv
    k64 = d["k"].double().repeat_interleave(r, dim=1)
    v64 = d["v"].double().repeat_interleave(r, dim=1)
    logits = torch.einsum("bhd,bhtd->bht", d["q"].double(), k64) * w.sm_scale
    ref = torch.einsum("bht,bhtd->bhd", torch.softmax(logits, dim=-1), v64)
    rot_off = akvq.K_PREROTATED | akvq.V_PREROTATED, akvq.Q_PREROTATED | akvq.OUT_ROTATED
    res = {}
    for name, rotate, salient in (("rotation + salient tokens (the method)", True, "psa"),
                                  ("rotation + text tokens salient", True, "tsa"),
                                  ("rotation only", True, None), ("salient tokens only", False, "psa"),
                                  ("plain 2-bit round-to-nearest", False, None)):
        cache = akvq.Cache(w.B, w.Hkv, w.G, t_cap, max(64, (w.n_text + 63) // 64 * 64))
        if salient == "psa":
            akvq.select_salient(cache, akvq.MODE_PSA, q_tail=d["q_tail"], k=d["k"], top_k=w.top_k, sm_scale=w.sm_scale)
        elif salient == "tsa":
            akvq.select_salient(cache, akvq.MODE_TSA, is_text=d["is_text"])
        akvq.quantize_append(cache, d["k"], d["v"], w.clip, flags=0 if rotate else rot_off[0])
        out, _ = akvq.decode_attention(cache, d["q"], w.sm_scale, flags=0 if rotate else rot_off[1])
        err = (out.double() - ref).norm(dim=-1) / ref.norm(dim=-1)
        res[name] = {"mean_rel_err": round(err.mean().item(), 4), "max_rel_err": round(err.max().item(), 4)}
    print(json.dumps({"metric": "decode-attention output error vs exact attention on unquantized K, V",
                      "workload": f"{w.name}(B={w.B})", "data": "synthetic", **res}))


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=100)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--workload", default="cfg2")
    ap.add_argument("--layers", type=int, default=0, help="override the number of layers (debugging)")
    ap.add_argument("--layer", type=int, default=-1, help="layer whose mode (TSA/PSA) a --phase run uses")
    ap.add_argument("--window", type=int, default=0,
                    help="--phase decode|quantize with a 16-bit recent window of this many rows (multiple of 64)")
    ap.add_argument("--tiered", action="store_true",
                    help="--phase decode|quantize with the 4-bit text tier (text tokens as row pairs, pivots 16-bit)")
    ap.add_argument("--rope", action="store_true",
                    help="--phase quantize with the rotary position embedding fused into the write path")
    ap.add_argument("--graph", action="store_true", help="--phase decode_step replayed as one HIP graph")
    ap.add_argument("--fused", action="store_true", help="--phase decode_step through akvq_decode_step (one launch per layer)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-extra-legs", action="store_true",
                    help="default line without the cfg3 / cfg5 decode legs and the streaming-read ceiling (profiling runs)")
    ap.add_argument("--n-split", type=int, default=0)
    ap.add_argument("--phase", default="all", choices=["all", "decode", "quantize", "select", "massive", "fold", "capacity", "ablation", "decode_step", "copy",
                             "stream", "oracle"],
                    help="time one call only (per-kernel studies; the default 'all' is the benchmark line)")
    ap.add_argument("--sets", type=int, default=0, help="distinct buffer sets to rotate through in --phase runs")
    ap.add_argument("--batch", type=int, default=0, help="override the workload's batch size (sweeps)")
    ap.add_argument("--budget-gb", type=float, default=256.0,
                    help="--phase capacity: HBM set aside for the KV cache of all layers together")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py: this build runs on ONE GPU only (no collectives, no sharding); use --gpus 1", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch
    from paper_2501_15021_amd import binding as akvq
    from paper_2501_15021_amd import synth

    akvq.lib()  # fail loudly if the HIP library is missing
    torch.cuda.set_device(0)
    w = synth.WORKLOADS[args.workload]
    if args.batch:
        import dataclasses
        w = dataclasses.replace(w, B=args.batch, name=f"{w.name}(B={args.batch})")
    if args.phase == "stream":
        print(json.dumps({"metric": "plain 128-bit streaming read (practical ceiling)",
                          **stream_ceiling(akvq, torch, warmup=max(args.warmup, 5), timed=max(args.steps, 40))}))
        return
    if args.phase == "oracle":
        return oracle_bench(args, w, synth, torch, np)
    if args.phase == "copy":
        # a plain device-to-device copy of known size: calibrates the HBM byte counters of rocprofv3 --pmc
        n = 1 << 30
        src = torch.empty(n, dtype=torch.uint8, device="cuda").random_(0, 255)
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        dst.copy_(src)
        e0.record()
        for _ in range(args.steps):
            dst.copy_(src)
        e1.record()
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / args.steps
        print(json.dumps({"metric": "plain copy", "bytes_read": n, "bytes_written": n, "ms_per_call": round(ms, 4),
                          "GBps_read_plus_write": round(2 * n / (ms * 1e-3) / 1e9, 1)}))
        return
    if args.phase == "massive":
        # pivot identification from massive activations on a synthetic residual stream (d_model 4096)
        d_model = 4096
        sets = []
        for i in range(2):
            d = synth.generate(w, layer=2 + 100 * i, device="cuda")
            hid = synth.hidden_states(w, d["pivots"].cpu(), d_model=d_model, layer=2 + 100 * i, device="cuda")
            sets.append((hid, akvq.Cache(w.B, w.Hkv, w.G, (w.T + 63) // 64 * 64, 64)))
            del d
        for i in range(args.warmup * 2):
            akvq.select_massive(sets[i % 2][1], sets[i % 2][0], 15, 100.0)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for i in range(args.steps * 2):
            akvq.select_massive(sets[i % 2][1], sets[i % 2][0], 15, 100.0)
        e1.record()
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / (args.steps * 2)
        nbytes = w.B * w.T * d_model * 2
        gbps = nbytes / (ms * 1e-3) / 1e9
        print(json.dumps({"metric": "select_massive call alone", "workload": w.name, "d_model": d_model,
                          "ms_per_call": round(ms, 5),
                          "roofline": {"bound": "hbm", "achieved": round(gbps, 1), "peak": HBM_PEAK_GBPS, "unit": "GB/s",
                                       "frac": round(gbps / HBM_PEAK_GBPS, 4), "traffic": None,
                                       "algorithmic_bytes_per_launch": nbytes}}))
        return
    if args.phase == "decode_step":
        return decode_step_bench(args, w, akvq, synth, torch, np)
    if args.phase == "ablation":
        return ablation_bench(args, w, akvq, synth, torch, np)
    if args.phase == "capacity":
        return capacity_bench(args, w, akvq, synth, torch, np)
    if args.phase == "fold":
        # offline fold of the rotation into one layer's W_V (output columns) and W_O (input rows), d_model 4096
        d_model = 4096
        g = torch.Generator(device="cuda").manual_seed(11)
        wv = (torch.randn(d_model, w.Hkv * 128, generator=g, device="cuda") / 64).half()
        wo = (torch.randn(w.Hq * 128, d_model, generator=g, device="cuda") / 64).half()
        ov, oo = torch.empty_like(wv), torch.empty_like(wo)
        res = {}
        for name, src, dst, axis in (("W_V columns", wv, ov, 1), ("W_O rows", wo, oo, 0)):
            for _ in range(args.warmup):
                akvq.fold_hadamard(src, axis, out=dst)
            torch.cuda.synchronize()
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(args.steps):
                akvq.fold_hadamard(src, axis, out=dst)
            e1.record()
            torch.cuda.synchronize()
            ms = e0.elapsed_time(e1) / args.steps
            nbytes = 2 * src.numel() * 2
            res[name] = {"shape": list(src.shape), "ms_per_call": round(ms, 5), "algorithmic_bytes": nbytes,
                         "GBps": round(nbytes / (ms * 1e-3) / 1e9, 1),
                         "frac_of_hbm_peak": round(nbytes / (ms * 1e-3) / 1e9 / HBM_PEAK_GBPS, 4)}
        print(json.dumps({"metric": "fold_hadamard call alone", "workload": w.name, "d_model": d_model, **res}))
        return
    if args.phase != "all":
        return phase_bench(args, w, akvq, synth, torch, np)
    L = args.layers or w.n_layers
    t_cap = (w.T + 63) // 64 * 64

    # ---- resident inputs and caches for every layer (distinct buffers: the 256 MB last-level cache cannot help) ----
    layers = []
    for layer in range(L):
        d = synth.generate(w, layer=layer, device="cuda")
        cache = akvq.Cache(w.B, w.Hkv, w.G, t_cap, w.s_cap(layer))
        layers.append((d, cache))
    torch.cuda.synchronize()

    ev = lambda: torch.cuda.Event(enable_timing=True)

    def step(events=None):
        for layer, (d, cache) in enumerate(layers):
            cache.T_len = 0
            if events is not None:
                e = [ev() for _ in range(4)]
                e[0].record()
            if w.mode(layer) == "tsa":
                akvq.select_salient(cache, akvq.MODE_TSA, is_text=d["is_text"])
            else:
                akvq.select_salient(cache, akvq.MODE_PSA, q_tail=d["q_tail"], k=d["k"], top_k=w.top_k,
                                    sm_scale=w.sm_scale)
            if events is not None:
                e[1].record()
            akvq.quantize_append(cache, d["k"], d["v"], w.clip)
            if events is not None:
                e[2].record()
            akvq.decode_attention(cache, d["q"], w.sm_scale, n_split=args.n_split)
            if events is not None:
                e[3].record()
                events.append((layer, e))

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    events = []
    t0 = time.perf_counter()
    for _ in range(args.steps):
        step(events)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    ms_per_step = wall * 1e3 / args.steps

    # ---- per-call durations from the HIP events recorded inside the timed region ----
    phase_ms = {"select": {}, "quantize": {}, "decode": {}}
    for layer, e in events:
        for i, name in enumerate(("select", "quantize", "decode")):
            phase_ms[name].setdefault(w.mode(layer), []).append(e[i].elapsed_time(e[i + 1]))
    tot = {name: sum(sum(v) for v in phase_ms[name].values()) / args.steps for name in phase_ms}
    kv_tokens = w.B * w.T * L
    bytes_l = [algorithmic_bytes(w, layer) for layer in range(L)]
    dec_bytes = sum(b["decode"] for b in bytes_l)
    q_bytes = sum(b["quantize"] for b in bytes_l)
    qin_bytes = sum(b["quantize_in"] for b in bytes_l)
    sel_bytes = sum(b["select"] for b in bytes_l)

    traffic_current = MEASURED_TRAFFIC["source_hash"] == kernel_source_hash()

    def roof(name, nbytes, ms, kernel):
        gbps = nbytes / (ms * 1e-3) / 1e9
        return {"kernel": kernel, "bound": "hbm", "achieved": round(gbps, 1), "peak": HBM_PEAK_GBPS, "unit": "GB/s",
                "frac": round(gbps / HBM_PEAK_GBPS, 4),
                "traffic": MEASURED_TRAFFIC.get(w.name, {}).get(name) if traffic_current else None,
                "avg_launch_ms": round(ms / L, 4), "algorithmic_bytes_per_launch": nbytes // L}

    rooflines = {
        "decode": roof("decode", dec_bytes, tot["decode"], "decode_mha_kernel/decode_gqa_kernel (+combine)"),
        "quantize": roof("quantize", q_bytes, tot["quantize"], "quantize_append_kernel (quantize_append_overlay_kernel in text-salient layers)"),
    }
    # quantize_append is bound by vector-instruction issue, not by HBM (counters: vector unit busy 97 % of the kernel):
    # the same launch against the vector peak without packed fp32 (256 CUs x 64 lanes x 2.4 GHz lane-operations/s),
    # counting the method's arithmetic only: per element 7 butterflies, one min/max step, three for the code
    # (multiply-add to an integer, clamp, pack).
    q_lane_ops = 11 * 2 * w.B * w.Hkv * w.T * 128 * L
    q_alu = q_lane_ops / (tot["quantize"] * 1e-3) / 1e9
    rooflines["quantize"]["alu"] = {"bound": "alu", "achieved": round(q_alu, 1), "peak": ALU_PEAK_GLANEOPS,
                                    "unit": "G lane-op/s", "frac": round(q_alu / ALU_PEAK_GLANEOPS, 4),
                                    "algorithmic_lane_ops_per_launch": q_lane_ops // L}
    if sel_bytes:
        rooflines["select"] = roof("select", sel_bytes, tot["select"], "psa_once_kernel or psa_row_stats_gqa_kernel+psa_mass_gqa_kernel (+topk)")
    dominant = max(("decode", "quantize", "select"), key=lambda n: tot[n])
    out = {
        "metric": METRIC,
        "value": kv_tokens / (tot["decode"] * 1e-3),
        "unit": "KV tokens/s (decode attention; whole-path and quantize rates in 'extra')",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(ms_per_step, 4),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "u2 codes; int8 and bf16 MFMA; f32 accumulate",
        "data": "synthetic (seeded; LLaVA-1.5-shaped prompt layout, outlier channels and pivot tokens planted)",
        "config": {"workload": f"{w.name}: {L} layers x B={w.B} x Hq={w.Hq}/Hkv={w.Hkv} x T={w.T}, G={w.G}, "
                               f"TSA layers {list(w.tsa_layers)}, PSA top-{w.top_k}, clip {w.clip}",
                   "step": "per layer: select_salient -> quantize_append(T rows) -> decode_attention(1 query/head)"},
        "roofline": rooflines[dominant if dominant in rooflines else "quantize"],
        "extra": {
            "whole_path_kv_tokens_per_s": kv_tokens / (ms_per_step * 1e-3),
            "ms_per_step_by_call": {k: round(v, 4) for k, v in tot.items()},
            "decode_GBps": rooflines["decode"]["achieved"], "decode_frac_of_hbm_peak": rooflines["decode"]["frac"],
            "quantize_input_GBps": round(qin_bytes / (tot["quantize"] * 1e-3) / 1e9, 1),
            "rooflines": rooflines,
            "decode_ms_per_layer": {m: round(float(np.mean(v)), 4) for m, v in phase_ms["decode"].items()},
            "quantize_ms_per_layer": {m: round(float(np.mean(v)), 4) for m, v in phase_ms["quantize"].items()},
            "select_ms_per_layer": {m: round(float(np.mean(v)), 4) for m, v in phase_ms["select"].items()},
            "call_ms_p10_median_p90": {
                name: {m: [round(float(x), 4) for x in np.percentile(v, (10, 50, 90))] for m, v in phase_ms[name].items()}
                for name in phase_ms},
            "n_split": args.n_split or akvq.lib().akvq_decode_default_splits(w.B, w.Hkv, w.T),
        },
    }
    if not args.no_cpu_baseline:
        layer = min(2, L - 1)
        base, oc = cpu_baseline(w, layer, layers[layer][0])
        out["cpu_baseline"] = base
        # the same layer on the GPU must agree with what the oracle just computed (sampled parity at full size)
        d, cache = layers[layer]
        out_gpu, _ = akvq.decode_attention(cache, d["q"], w.sm_scale, n_split=args.n_split)
        ref, _ = oc.decode(d["q"].cpu().numpy(), w.sm_scale)
        same_sets = bool(np.array_equal(cache.sal_idx.cpu().numpy(), oc.sal_idx))
        codes_equal = same_sets and bool(np.array_equal(cache.k_codes.cpu().numpy().view(np.uint32), oc.k_codes)
                                         and np.array_equal(cache.v_codes.cpu().numpy().view(np.uint32), oc.v_codes))
        err = np.abs(out_gpu.cpu().numpy() - ref).max(-1) / np.abs(ref).max(-1)
        out["extra"]["parity_vs_oracle_on_baseline_layer"] = {
            "salient_sets_equal": same_sets, "codes_bit_exact": codes_equal,
            "attention_max_rel_err": float(err.max()) if same_sets else None}
        if oc.margins is not None:   # how far the oracle's fp64 masses are from a tie at the selection boundary
            differ = int((cache.sal_idx.cpu().numpy() != oc.sal_idx).any(axis=-1).sum())
            out["extra"]["parity_vs_oracle_on_baseline_layer"].update({
                "units": int(oc.margins.size), "units_whose_set_differs": differ,
                "min_margin": float(oc.margins.min()), "units_with_margin_below_1e-4": int((oc.margins < 1e-4).sum()),
                "units_with_margin_below_1e-3": int((oc.margins < 1e-3).sum())})
    if not args.no_extra_legs and w.name == "cfg2" and not args.layers and not args.batch:
        # the long-context configurations the target is quoted on, and the practical ceiling, in the same run
        del layers, d, cache
        torch.cuda.empty_cache()
        for name in ("cfg3", "cfg5"):
            out["extra"]["rooflines"][f"decode_{name}"] = decode_alone(synth.WORKLOADS[name], akvq, synth, torch, np)
            torch.cuda.empty_cache()
        # the prefill configuration (write path + pivot selection at 16384 tokens) and the grouped-query one
        for name in ("cfg4", "cfg5"):
            out["extra"][f"prefill_{name}"] = prefill_alone(synth.WORKLOADS[name], akvq, synth, torch, np)
            torch.cuda.empty_cache()
        sc = stream_ceiling(akvq, torch)
        out["extra"]["stream_ceiling_GBps"] = sc["GBps"]
        out["extra"]["stream_ceiling"] = sc
    print(json.dumps(out))


if __name__ == "__main__":
    main()
