#!/usr/bin/env python3
"""Benchmark: cache tokens compacted per second per layer on one MI355X.

One step = one still_compact_model call over every layer of the workload (the
whole hot path: RoPE-fix staging, cross-attention, self-attention, FFN, output
heads, re-rotation) with inputs already resident in HBM.  Prints one JSON line.

The headline workload is the 36-layer Qwen-8B-shaped 8k -> 1024 stack; the
128k -> 655 (200x) stack follows by default under "workloads", measured the
same way after the headline's buffers are freed.

The dominant kernel (flash cross-attention) is timed live with hipEvent pairs
on its launch stream during the timed region; its algorithmic FLOPs per launch
(QK^T and P.X for all KV heads x cross heads of one layer) divided by the
average launch duration gives the roofline point.  The KV-stream kernel
(RoPE-fix staging, the one HBM-bound step) is timed the same way against the
HBM peak.  The fp64 oracle is timed on a bounded sample (KV heads of one
layer, about 25 s per workload) as a CPU baseline.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_FP16_TFLOPS = 2500.0     # MI355X dense fp16/bf16 MFMA
PEAK_HBM_GBS = 8000.0

# HBM bytes per launch of the cross-attention kernel on the default workload,
# from rocprofv3 PMC FETCH_SIZE / WRITE_SIZE passes scaled by what the same
# counters read for a 1 GiB device copy (factors 2.0 and 1.0).  Valid only for
# the kernel sources with this digest; any later change reports null.
MEASURED_TRAFFIC = {"workload": 2, "sources_sha256_16": "6b0dc2a751f8d041", "bytes_per_launch": 3636593766}
KERNEL_SOURCES = tuple(f"paper_2606_07878_amd/csrc/{f}" for f in ("attn.hpp", "common.hpp", "host.hpp", "xattn.hip"))


def measured_traffic(workload_id: int):
    import hashlib
    h = hashlib.sha256()
    for f in KERNEL_SOURCES:
        with open(os.path.join(ROOT, f), "rb") as fh:
            h.update(fh.read())
    if workload_id != MEASURED_TRAFFIC["workload"] or h.hexdigest()[:16] != MEASURED_TRAFFIC["sources_sha256_16"]:
        return None
    return MEASURED_TRAFFIC["bytes_per_launch"]


def ca_flops_per_launch(w, N=None) -> float:
    c = w.cfg
    per_pair = 2.0 * w.t * (N or w.n_tokens) * (c.dc + 2 * c.head_dim)
    return per_pair * c.n_kv_heads * c.n_cross_heads


def layer_flops(w, N=None) -> float:
    """Algorithmic FLOPs of one layer (cheapest exact association)."""
    c = w.cfg
    N = N or w.n_tokens
    H, t, D, d, nc, dc, ns, ds, F = (c.n_kv_heads, w.t, c.latent_dim, c.head_dim, c.n_cross_heads, c.dc,
                                     c.n_self_heads, c.ds, c.ffn_hidden)
    Ht = H * t
    f = 2.0 * Ht * D * nc * dc                          # Q projection
    f += 2.0 * H * N * 2 * d * nc * dc                  # K projection
    f += 2.0 * H * nc * t * N * (dc + 2 * d)            # QK^T and P.X
    f += 2.0 * Ht * 2 * d * nc * dc                     # (P X) W_V
    f += 2.0 * Ht * nc * dc * D                         # W_O
    if ns:
        f += 2.0 * Ht * D * 3 * ns * ds + 2.0 * H * ns * t * t * 2 * ds + 2.0 * Ht * ns * ds * D
    if c.ffn_kind == 1:
        f += 2.0 * Ht * D * 3 * F
    elif c.ffn_kind == 2:
        f += 2.0 * Ht * D * 2 * F
    f += 2.0 * Ht * D * 2 * d                           # output heads
    return f


def cpu_baseline(w, budget_s: float = 25.0) -> dict:
    """Time the fp64 oracle (numpy, all BLAS threads) on layer 0, one KV head
    after another, until every head is done or the budget is spent."""
    import numpy as np
    from oracle import compactor
    from paper_2606_07878_amd import synth
    try:
        from threadpoolctl import threadpool_info
        threads = max([i.get("num_threads", 0) for i in threadpool_info() if i.get("user_api") == "blas"] or [0])
    except Exception:
        threads = 0
    cache = synth.as_f64(synth.make_cache(w, 0))
    wts = synth.as_f64(synth.make_weights(w, 0))
    H = w.cfg.n_kv_heads
    done, dt = 0, 0.0
    while done < H and dt < budget_s:
        t0 = time.perf_counter()
        compactor.compact_layer(cache["K"], cache["V"], cache["positions"], w.rope_theta, wts, w.cfg, w.t,
                                heads=[done])
        dt += time.perf_counter() - t0
        done += 1
    per_layer = dt / done * H
    sample = (f"fp64 oracle, layer 0, KV heads 0..{done - 1} of {H} ({dt:.1f} s)"
              + ("" if done == H else f", scaled x{H / done:g} to one layer"))
    return {"value": round(w.n_tokens / per_layer, 1), "unit": "tokens/s/layer",
            "cores": int(threads or os.cpu_count()), "kind": "oracle", "sample": sample}


def copy_probe(mib: int, dev) -> None:
    """One plain device-to-device copy of a known size; its FETCH_SIZE/WRITE_SIZE
    counters calibrate what the same counters read for the compactor kernels."""
    import torch
    n = mib << 20
    src = torch.ones(n, dtype=torch.uint8, device=dev)
    dst = torch.empty_like(src)
    torch.cuda.synchronize()
    dst.copy_(src)
    torch.cuda.synchronize()
    print(f"[bench] copy probe: {mib} MiB read + {mib} MiB written", file=sys.stderr, flush=True)
    del src, dst


# MI355X: 8 XCDs (GRBM_GUI_ACTIVE is summed over them), 1024 SIMDs
N_XCD, N_SIMD = 8, 1024


def summarize_counters(path: str, top: int = 400) -> None:
    """Per-kernel means of a rocprofv3 counter-collection CSV (one row per
    dispatch and counter), with the derived figures used in the profiles:
    MFMA busy fraction = SQ_VALU_MFMA_BUSY_CYCLES / (GRBM_GUI_ACTIVE / 8 x 1024),
    f16 MFMA rate = SQ_INSTS_VALU_MFMA_MOPS_F16 x 512 flops per dispatch time,
    DRAM bytes read = TCC_EA0_RDREQ_DRAM_32B x 32, written = TCC_EA0_WRREQ_DRAM x 64,
    FETCH_SIZE / WRITE_SIZE in KiB as counted."""
    import collections
    import csv
    import re
    acc = collections.defaultdict(lambda: collections.defaultdict(float))
    disp = collections.defaultdict(set)
    dur = collections.defaultdict(dict)
    with open(path) as f:
        for r in csv.DictReader(f):
            name = re.sub(r"\(.*", "", r["Kernel_Name"])[:96] + f" grid={r['Grid_Size']}"
            disp[name].add(r["Dispatch_Id"])
            acc[name][r["Counter_Name"]] += float(r["Counter_Value"])
            dur[name][r["Dispatch_Id"]] = int(r["End_Timestamp"]) - int(r["Start_Timestamp"])
    order = sorted(acc, key=lambda k: -sum(dur[k].values()))[:top]
    for name in order:
        n = len(disp[name])
        m = {c: v / n for c, v in acc[name].items()}
        us = sum(dur[name].values()) / n / 1e3
        parts = [f"n={n}", f"avg_us={us:.1f}"]
        if "GRBM_GUI_ACTIVE" in m and "SQ_VALU_MFMA_BUSY_CYCLES" in m:
            parts.append(f"mfma_busy={m['SQ_VALU_MFMA_BUSY_CYCLES'] / (m['GRBM_GUI_ACTIVE'] / N_XCD * N_SIMD):.3f}")
        if "SQ_INSTS_VALU_MFMA_MOPS_F16" in m and us > 0:
            parts.append(f"f16_TFLOPs={m['SQ_INSTS_VALU_MFMA_MOPS_F16'] * 512 / us * 1e-6:.1f}")
        if "SQ_LDS_IDX_ACTIVE" in m and "SQ_LDS_BANK_CONFLICT" in m and m["SQ_LDS_IDX_ACTIVE"] > 0:
            parts.append(f"lds_conflict_frac={m['SQ_LDS_BANK_CONFLICT'] / m['SQ_LDS_IDX_ACTIVE']:.3f}")
        if "TCC_EA0_RDREQ_DRAM_32B" in m:
            rd = m["TCC_EA0_RDREQ_DRAM_32B"] * 32
            parts.append(f"dram_read_MB={rd / 1e6:.1f} ({rd / us * 1e-6:.2f} TB/s)")
        if "TCC_EA0_WRREQ_DRAM" in m:
            wr = m["TCC_EA0_WRREQ_DRAM"] * 64
            parts.append(f"dram_write_MB={wr / 1e6:.1f} ({wr / us * 1e-6:.2f} TB/s)")
        for c in ("FETCH_SIZE", "WRITE_SIZE"):
            if c in m:
                parts.append(f"{c}_KiB={m[c]:.1f}")
        print(f"{name} | " + " ".join(parts))


def consumer_attend(w, Ck, Cv, Ks, Vs, dev, binding, reps: int = 20, suffix: int = 64) -> dict:
    """One decode step of the base model's attention over every layer
    (query_group query heads per KV head, one query each): over the compact
    cache [C_k; 64 suffix tokens] with a bias, and over the full uncompacted
    cache [K; 64 suffix tokens].  The L calls of a step are captured in one
    HIP graph (as a decode step would run) and the graph is replayed; the time
    per layer is graph time / L, so launch gaps inside the graph count, host
    launch costs do not.  Bytes are the algorithmic K and V stream (each entry
    read once)."""
    import torch
    from paper_2606_07878_amd import configs
    cfg = w.cfg
    H, d, g, L = cfg.n_kv_heads, cfg.head_dim, w.query_group, len(Ck)
    gen = torch.Generator(device=dev)
    gen.manual_seed(12345)
    q = torch.randn(H * g, 1, d, generator=gen, device=dev).to(torch.bfloat16)
    Ks_sfx = torch.randn(H, suffix, d, generator=gen, device=dev).to(torch.bfloat16)
    Vs_sfx = torch.randn(H, suffix, d, generator=gen, device=dev).to(torch.bfloat16)
    beta = torch.randn(H, w.t, generator=gen, device=dev)
    ws = torch.empty(binding.still_attend_workspace_size(binding.still_attend_config(
        H, g, d, 1, 0, w.n_tokens + suffix, 0, 0.0, configs.MODE_BF16)), dtype=torch.uint8, device=dev)
    full_k = [torch.cat([K, Ks_sfx], dim=1) for K in Ks]
    full_v = [torch.cat([V, Vs_sfx], dim=1) for V in Vs]
    res = {}
    for name, args in (("compact", lambda l: (Ck[l], Cv[l], beta, Ks_sfx, Vs_sfx)),
                       ("full", lambda l: (None, None, None, full_k[l], full_v[l]))):
        outs = [torch.empty_like(q) for _ in range(L)]

        def step():
            for l in range(L):
                binding.attend(q, *args(l), group=g, workspace=ws, out=outs[l])
        step()                                   # eager warm-up (first-launch costs)
        torch.cuda.synchronize()
        s = torch.cuda.Stream(device=dev)
        s.wait_stream(torch.cuda.current_stream(dev))
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.stream(s):
            with torch.cuda.graph(graph, stream=s):
                step()
        torch.cuda.current_stream(dev).wait_stream(s)
        graph.replay()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            graph.replay()
        e1.record()
        torch.cuda.synchronize()
        us = e0.elapsed_time(e1) * 1e3 / (reps * L)
        entries = (w.t + suffix) if name == "compact" else (w.n_tokens + suffix)
        nbytes = H * entries * d * 2 * 2
        res[name] = {"entries": entries, "us_per_layer": round(us, 3), "bytes": nbytes,
                     "GB_s": round(nbytes / (us * 1e-6) / 1e9, 1),
                     "hbm_frac": round(nbytes / (us * 1e-6) / 1e9 / PEAK_HBM_GBS, 4)}
        del graph
    res["decode_speedup"] = round(res["full"]["us_per_layer"] / res["compact"]["us_per_layer"], 2)
    res["shape"] = {"H_kv": H, "query_group": g, "n_queries": 1, "d": d, "suffix": suffix, "io": "bf16",
                    "timing": "HIP graph of the L layer calls, replayed"}
    return res


def backward_measure(wid: int, dev, binding, reps: int = 3, N: int = 8192, t: int = 256) -> dict:
    """One layer of the compactor backward pass (still_compact_layer_backward,
    fp32 mode: forward with saved activations, then the reverse sweep) at
    the workload's compactor shape on an N-token cache compacted to t.
    Algorithmic FLOPs: three times the forward layer's (the forward itself,
    then one product each for the input and the weight gradients)."""
    import torch
    from paper_2606_07878_amd import configs, synth
    w = configs.shrink(configs.get_workload(wid), n_tokens=N, t=t)
    K, V, pos, W = synth.make_layer_torch(w, 0, dev, dtype=torch.float32)
    gen = torch.Generator(device=dev)
    gen.manual_seed(99)
    dCk = torch.randn(w.cfg.n_kv_heads, t, w.cfg.head_dim, generator=gen, device=dev)
    dCv = torch.randn(w.cfg.n_kv_heads, t, w.cfg.head_dim, generator=gen, device=dev)
    ccfg = binding.make_config(w.cfg, configs.MODE_FP32)
    ws = torch.empty(binding.still_backward_workspace_size(ccfg, N, t), dtype=torch.uint8, device=dev)
    binding.compact_layer_backward(w.cfg, W, K, V, pos, w.rope_theta, t, dCk, dCv, workspace=ws)   # warm-up
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(reps):
        binding.compact_layer_backward(w.cfg, W, K, V, pos, w.rope_theta, t, dCk, dCv, workspace=ws)
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / reps
    flops = 3.0 * layer_flops(w, N)
    return {"workload": f"{w.name}, backward of one layer, N {N} -> t {t}, fp32 mode", "ms_per_layer": round(ms, 3),
            "reps": reps, "algorithmic_tflop": round(flops * 1e-12, 4),
            "achieved_tflops": round(flops / (ms * 1e-3) * 1e-12, 2),
            "frac_of_fp32_mfma_peak": round(flops / (ms * 1e-3) / 157.3e12, 4)}


def kv_stream_bytes(w, N=None) -> dict:
    """Bytes of the RoPE-fix staging kernel per layer: the KV cache read once
    (the algorithmic stream) and the fp16 X / X^T copies it writes."""
    c = w.cfg
    N = N or w.n_tokens
    npad = -(-N // 256) * 256
    read = 2 * c.n_kv_heads * N * c.head_dim * 2
    write = c.n_kv_heads * N * 2 * c.head_dim * 2 + c.n_kv_heads * 2 * c.head_dim * npad * 2
    return {"read": read, "write": write}


def run_workload(wid: int, steps: int, warmup: int, dev, binding, consumer: bool = False) -> dict:
    """Generate a workload's stack on the device, time `steps` whole steps
    after `warmup` untimed ones, and return its measurements.  The dominant
    kernel (cross-attention) and the KV-stream kernel (RoPE-fix staging) are
    timed live with hipEvent pairs on their launch stream inside the timed
    region."""
    import torch
    from paper_2606_07878_amd import configs, synth

    w = configs.get_workload(wid)
    L = w.n_layers
    print(f"[bench] generating {L} layers of {w.name}", file=sys.stderr, flush=True)
    Ks, Vs, Ws = [], [], []
    pos = None
    for l in range(L):
        K, V, pos, W = synth.make_layer_torch(w, l, dev)
        Ks.append(K)
        Vs.append(V)
        Ws.append(binding.LayerWeights(w.cfg, W))
    ccfg = binding.make_config(w.cfg, configs.MODE_BF16)
    N, t = w.n_tokens, w.t
    ws_bytes = binding.still_workspace_size(ccfg, N, t, L)
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device=dev)
    Ck = [torch.empty(w.cfg.n_kv_heads, t, w.cfg.head_dim, dtype=torch.bfloat16, device=dev) for _ in range(L)]
    Cv = [torch.empty_like(c) for c in Ck]
    outp = torch.empty(t, dtype=torch.float64, device=dev)
    stream = torch.cuda.current_stream(dev)

    # Iterative workloads: each round appends fresh tokens to the compact cache
    # of the previous call and recompacts to t.  The fresh tokens of every
    # round sit pre-generated behind a t-row slot that takes the previous C_k,
    # C_v (a device copy); positions likewise.
    R, Fr = w.rounds, w.fresh_tokens
    Kr, Vr, Pr = [], [], []
    for r in range(R):
        T0 = N + r * Fr
        fpos = torch.arange(T0, T0 + Fr, dtype=torch.float64, device=dev)
        kl, vl = [], []
        for l in range(L):
            Kf, Vf, _, _ = synth.make_layer_torch(w, 1000 * (r + 1) + l, dev, n_tokens=Fr, positions=fpos,
                                                   weights=False)
            kb = torch.empty(w.cfg.n_kv_heads, t + Fr, w.cfg.head_dim, dtype=torch.bfloat16, device=dev)
            vb = torch.empty_like(kb)
            kb[:, t:] = Kf
            vb[:, t:] = Vf
            kl.append(kb)
            vl.append(vb)
        pb = torch.empty(t + Fr, dtype=torch.float64, device=dev)
        pb[t:] = fpos
        Kr.append(kl)
        Vr.append(vl)
        Pr.append(pb)
    if R:
        print(f"[bench] {R} rounds of {Fr} fresh tokens per layer prepared", file=sys.stderr, flush=True)

    def call(Kin, Vin, p, n):
        st = binding.still_compact_model(ccfg, Ws, Kin, Vin, p, n, w.rope_theta, t, binding.STILL_F_REROTATE,
                                         Ck, Cv, outp, ws, ws_bytes, stream.cuda_stream)
        if st != 0:
            raise binding.StillError(st, binding.still_last_error())

    def step():
        call(Ks, Vs, pos, N)
        for r in range(R):
            for l in range(L):
                Kr[r][l][:, :t].copy_(Ck[l])
                Vr[r][l][:, :t].copy_(Cv[l])
            Pr[r][:t].copy_(outp)
            call(Kr[r], Vr[r], Pr[r], t + Fr)

    for i in range(warmup):
        step()
        torch.cuda.synchronize()
        print(f"[bench] warmup {i + 1}/{warmup} done", file=sys.stderr, flush=True)
    kc = binding.KERNEL_CLASSES
    binding.still_timing_reset()
    binding.still_timing_enable((1 << kc["cross_attn"]) | (1 << kc["stage"]))
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    e0.record(stream)
    for i in range(steps):
        step()
    e1.record(stream)
    torch.cuda.synchronize()
    binding.still_timing_enable(0)
    ms_step = e0.elapsed_time(e1) / steps
    att_ms, att_n = binding.still_timing_read(kc["cross_attn"])
    stg_ms, stg_n = binding.still_timing_read(kc["stage"])
    print(f"[bench] {w.name}: {steps} steps, {ms_step:.2f} ms/step", file=sys.stderr, flush=True)

    # per-class breakdown (separate, untimed pass)
    binding.still_timing_reset()
    binding.still_timing_enable((1 << len(kc)) - 1)
    step()
    torch.cuda.synchronize()
    binding.still_timing_enable(0)
    breakdown = {}
    for name, cls in kc.items():
        ms, n = binding.still_timing_read(cls)
        if n:
            breakdown[name] = round(ms / L, 4)
    binding.still_timing_reset()

    cons = consumer_attend(w, Ck, Cv, Ks, Vs, dev, binding) if consumer else None

    tokens_in = N + R * (t + Fr)                        # cache tokens entering the calls of one step
    tokens_per_s_layer = tokens_in * L / (ms_step / 1e3)
    avg_att_s = att_ms / att_n / 1e3
    launch_flops = (ca_flops_per_launch(w) + R * ca_flops_per_launch(w, t + Fr)) / (1 + R)
    achieved = launch_flops / avg_att_s / 1e12
    kvb = [kv_stream_bytes(w)] + [kv_stream_bytes(w, t + Fr)] * R
    kv_read = sum(b["read"] for b in kvb) / len(kvb)
    kv_moved = sum(b["read"] + b["write"] for b in kvb) / len(kvb)
    avg_stg_s = stg_ms / stg_n / 1e3
    res = {
        "value": round(tokens_per_s_layer, 1),
        "ms_per_step": round(ms_step, 3),
        "ms_per_layer": round(ms_step / L, 4),
        "config": {"workload": w.name, "layers": L, "N": N, "t": t, "rounds": R, "fresh_per_round": Fr,
                   "H_kv": w.cfg.n_kv_heads,
                   "d": w.cfg.head_dim, "D": w.cfg.latent_dim, "n_cross": w.cfg.n_cross_heads,
                   "n_self": w.cfg.n_self_heads, "ffn_hidden": w.cfg.ffn_hidden, "io": "bf16",
                   "parallelism": "single-gpu"},
        "roofline": {"bound": "mfma", "kernel": "cross_attn", "achieved": round(achieved, 2),
                     "peak": PEAK_FP16_TFLOPS, "unit": "TFLOP/s", "frac": round(achieved / PEAK_FP16_TFLOPS, 4),
                     "traffic": measured_traffic(wid), "traffic_unit": "bytes/launch",
                     "avg_launch_ms": round(avg_att_s * 1e3, 4),
                     "launches": att_n,
                     "flops_per_launch": launch_flops},
        "kv_stream": {"bound": "hbm", "kernel": "stage_x (RoPE-fix staging)", "unit": "GB/s",
                      "peak": PEAK_HBM_GBS, "avg_launch_ms": round(avg_stg_s * 1e3, 4), "launches": stg_n,
                      "algorithmic_bytes": kv_read, "achieved": round(kv_read / avg_stg_s / 1e9, 1),
                      "frac": round(kv_read / avg_stg_s / 1e9 / PEAK_HBM_GBS, 4),
                      "moved_bytes": kv_moved, "moved_GB_s": round(kv_moved / avg_stg_s / 1e9, 1),
                      "moved_frac": round(kv_moved / avg_stg_s / 1e9 / PEAK_HBM_GBS, 4)},
        "layer_mfma_frac": round((layer_flops(w) + R * layer_flops(w, t + Fr)) / (ms_step / L / 1e3) / 1e12
                                 / PEAK_FP16_TFLOPS, 4),
        "kernel_ms_per_layer": breakdown,
    }
    if cons is not None:
        res["consumer_attend"] = cons
    del Ks, Vs, Ws, ws, Ck, Cv, Kr, Vr, Pr
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return res


def library_gemm_reference(wid: int, dev, reps: int = 20) -> dict:
    """The vendor library's fp16 product (torch.bmm, C = A B with B given as
    the transpose of a row-major [N][K] operand, fp32 accumulation) timed on
    the latent-side product shapes of one workload: the practical MFMA rate of
    the chip on those shapes, for comparison with this library's kernels."""
    import torch
    from paper_2606_07878_amd import configs
    w = configs.get_workload(wid)
    c = w.cfg
    H, t = c.n_kv_heads, w.t
    shapes = {   # name: (batch, M, N, K)
        "self q/k/v projection": (1, H * t, c.n_self_heads * c.ds, c.latent_dim),
        "cross q projection": (1, H * t, c.n_cross_heads * c.dc, c.latent_dim),
        "cross output W_O": (1, H * t, c.latent_dim, c.n_cross_heads * c.dc),
        "FFN gate+up": (1, H * t, 2 * c.ffn_hidden, c.latent_dim),
        "FFN down": (1, H * t, c.latent_dim, c.ffn_hidden),
        "self logits (per head)": (H * c.n_self_heads, t, t, c.ds),
        "self P v (per head)": (H * c.n_self_heads, t, c.ds, t),
        "(P X) W_V": (1, H * c.n_cross_heads * t, c.dc, 2 * c.head_dim),
    }
    out = {}
    for name, (b, M, N, K) in shapes.items():
        a = torch.randn(b, M, K, device=dev, dtype=torch.float16)
        bt = torch.randn(b, N, K, device=dev, dtype=torch.float16).transpose(1, 2).contiguous()
        for _ in range(3):
            torch.bmm(a, bt)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            torch.bmm(a, bt)
        e1.record()
        torch.cuda.synchronize()
        us = e0.elapsed_time(e1) / reps * 1e3
        fl = 2.0 * b * M * N * K
        out[name] = {"batch": b, "M": M, "N": N, "K": K, "us": round(us, 1), "tflops": round(fl / us * 1e-6, 1),
                     "frac_of_2.5PF": round(fl / us * 1e-6 / 2500.0, 3)}
        print(f"[gemm-ref] {name:24s} {b}x{M}x{N}x{K}: {us:8.1f} us {fl / us * 1e-6:7.1f} TFLOP/s", flush=True)
        del a, bt
    torch.cuda.empty_cache()
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--workload", type=int, default=2, help="registered workload id (default: 8k/8x Qwen-8B stack)")
    ap.add_argument("--extra-workloads", default="4",
                    help="comma-separated workload ids also measured after the headline one, each reported "
                         "under 'workloads' (default: 4, the 128k/200x stack; '' for none)")
    ap.add_argument("--extra-steps", type=int, default=3)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--copy-probe-mib", type=int, default=0,
                    help="run one plain device copy of this many MiB first (HBM counter calibration)")
    ap.add_argument("--no-backward", action="store_true", help="skip the backward-pass measurement")
    ap.add_argument("--no-consumer", action="store_true",
                    help="skip the decode-attention measurement (shorter profiler runs)")
    ap.add_argument("--summarize-counters", metavar="CSV",
                    help="print per-kernel means of a rocprofv3 counter-collection CSV and exit (no GPU use)")
    ap.add_argument("--backward-only", action="store_true",
                    help="time only the backward pass of one layer (the 'backward' object) and print that object")
    ap.add_argument("--library-gemm-reference", action="store_true",
                    help="time the vendor library's fp16 product (torch.bmm) on the latent-side product shapes "
                         "of --workload and print that object (reference for the MFMA rate, no compaction)")
    ap.add_argument("--consumer-only", action="store_true",
                    help="time only the decode attention over the compacted and the full cache (after one "
                         "compaction step) and print that object")
    args = ap.parse_args()
    if args.summarize_counters:
        summarize_counters(args.summarize_counters)
        return
    if args.gpus != 1:
        print(f"bench.py measures one GPU only (got --gpus {args.gpus}): the library runs a layer on one "
              "MI355X and has no multi-GPU path; a layer's KV heads or the layers of a stack would be "
              "spread over GPUs by the caller.", file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_2606_07878_amd import binding, configs

    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    if args.copy_probe_mib:
        copy_probe(args.copy_probe_mib, dev)
    if args.backward_only:
        print(json.dumps({"backward": backward_measure(args.workload, dev, binding)}), flush=True)
        return
    if args.library_gemm_reference:
        w = configs.get_workload(args.workload)
        print(json.dumps({"library_gemm_reference": library_gemm_reference(args.workload, dev),
                          "config": {"workload": w.name}}), flush=True)
        return
    if args.consumer_only:
        w = configs.get_workload(args.workload)
        res = run_workload(args.workload, 1, args.warmup, dev, binding, consumer=True)
        print(json.dumps({"consumer_attend": res["consumer_attend"], "config": {"workload": w.name}}), flush=True)
        return
    head = run_workload(args.workload, args.steps, args.warmup, dev, binding, consumer=not args.no_consumer)
    extras = [int(x) for x in args.extra_workloads.split(",") if x.strip() and int(x) != args.workload]
    workloads = {}
    for wid in extras:
        r = run_workload(wid, args.extra_steps, 1, dev, binding)
        r.update({"steps": args.extra_steps, "warmup": 1, "unit": "tokens/s/layer"})
        workloads[f"workload_{wid}"] = r
    out = {
        "metric": "cache tokens compacted/sec/layer + % HBM BW or % MFMA peak, 1 MI355X",
        "value": head["value"],
        "unit": "tokens/s/layer",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": head["ms_per_step"],
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f16", "data": "synthetic",
    }
    out.update({k: v for k, v in head.items() if k not in ("value", "ms_per_step")})
    if workloads:
        out["workloads"] = workloads
    if not args.no_backward:
        print("[bench] timing the backward pass", file=sys.stderr, flush=True)
        out["backward"] = backward_measure(args.workload, dev, binding)
    if not args.no_cpu_baseline:
        print("[bench] timing the CPU oracle on bounded samples", file=sys.stderr, flush=True)
        out["cpu_baseline"] = cpu_baseline(configs.get_workload(args.workload))
        for wid in extras:
            out["workloads"][f"workload_{wid}"]["cpu_baseline"] = cpu_baseline(configs.get_workload(wid))
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
