#!/usr/bin/env python3
"""Benchmark of the W4A8 linear layer on one MI355X.

A step = one decode pass over all 224 projections of a LLaMA-7B-shaped model
(32 blocks x q/k/v/o/gate/up/down), run once for each token count M in
{1, 4, 16}, with the activation quantizer fused as prologue and the per-channel
dequantisation as epilogue.  Projections that read the same activation (q/k/v,
gate/up) go through agq_gemm_w4a8_multi, i.e. one kernel launch: 4 launches per
block, 384 per step.  All 224 packed 4-bit
weight matrices are distinct buffers (3.24 GB, far beyond the 256 MB Infinity
Cache), resident in HBM before the timed region.  The metric is the algorithmic
bytes of those calls (4-bit weights + fp16 scales + fp16 activation in and out)
per second.

The same line also carries the same sweep with 4-bit activations (W4A4), the
prefill regime (M = 2048, the seven shapes of one block, W4A8 and W4A4) as int8
TOP/s, the TRIP layer on the same shapes beside the plain one, the attention
block at LLaMA-13B size (from fp16 probabilities, and from int8 Q and K in one
kernel) with pruning, one whole block of the pipeline (RMSNorm, projections,
rotary embedding, attention, pruning, MLP) at LLaMA-13B and 7B shapes, a stack of
four such blocks with the cascade schedule of Eq.9, the
roofline of the dominant kernel, and the CPU oracle timed on the host cores.
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

HBM_PEAK_GBS = 8000.0          # MI355X HBM3E
F16_PEAK_TFLOPS = 2500.0   # dense fp16 MFMA
INT8_PEAK_TOPS = 5000.0        # MI355X dense int8 MFMA
DECODE_M = (1, 4, 16)
PREFILL_M = 2048

# HBM traffic per launch from rocprofv3 --pmc runs of this file (FETCH_SIZE x 2.0 KiB + WRITE_SIZE x 1.0 KiB, the
# factors a 256 MiB copy gives).  A counter run cannot happen inside a timed run, so the figures are carried here
# from the summaries under profiles/, each with the digest of the kernel source it was measured on: when that
# source has changed since, the figure is reported as null (stale) instead of a number that no longer holds.
#   name: (bytes per launch, profiles/ file, source file, first 12 hex digits of the source's sha256)
MEASURED_TRAFFIC = {
    "decode": (26.3e6, "profiles/gemm_decode_llama7b_sweep.md", "agq_gemm_decode.hip", "b749db6894b5"),
    "attn": (252.6e6, "profiles/log2_attn_llama13b_block.md", "agq_attn.hip", "e21c65f1ff1e"),
    "tiled": (186.2e6, "profiles/gemm_decode_llama7b_sweep.md", "agq_gemm_tiled.hip", "c80578732a47"),
}


def measured_traffic(name):
    """(bytes or None, note) for the roofline objects."""
    import hashlib
    nbytes, prof, src, digest = MEASURED_TRAFFIC[name]
    path = os.path.join(ROOT, "paper_2312_05693_amd", "csrc", src)
    now = hashlib.sha256(open(path, "rb").read()).hexdigest()[:12]
    if now != digest:
        return None, "stale: %s changed since the counter run summarised in %s" % (src, prof)
    return nbytes, "rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE, %s" % prof


def algorithmic_bytes(M, K, N):
    """4-bit weights + fp16 weight scales + fp16 activation in + fp16 out."""
    return K * N // 2 + 2 * N + 2 * M * K + 2 * M * N


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=30)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-prefill", action="store_true")
    ap.add_argument("--no-attention", action="store_true")
    ap.add_argument("--no-trip", action="store_true")
    ap.add_argument("--no-block", action="store_true")
    ap.add_argument("--no-chain", action="store_true", help="skip the one-launch chain of the decode pass")
    ap.add_argument("--no-probe", action="store_true", help="skip the plain-read / empty-kernel probe of the device")
    ap.add_argument("--no-by-m", action="store_true", help="skip the sweep over 32..1024 rows in the prefill section")
    ap.add_argument("--copy-probe", action="store_true",
                    help="also run a 256 MiB device copy: the known traffic that scales the FETCH_SIZE / WRITE_SIZE counters")
    ap.add_argument("--per-projection", action="store_true", help="seven single calls per block instead of four")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build runs on one GPU only (the path has no collective); use --gpus 1", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch
    from paper_2312_05693_amd import binding as agq, synth

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    torch.cuda.set_device(0)
    agq.lib()
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(1)

    if args.copy_probe:
        src = torch.empty(256 << 20, dtype=torch.uint8, device=dev).fill_(7)
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst

    def make_packed(N, K):
        """N(0, 0.02) weights -> symmetric 4-bit per output channel -> packed blob (all on the GPU; input recipe)."""
        w = torch.randn((N, K), generator=gen, device=dev, dtype=torch.float32) * 0.02
        sw = (w.abs().amax(dim=1) / 7.0).to(torch.float16)
        sw = torch.where(sw == 0, torch.ones_like(sw), sw)
        wq = torch.clamp(torch.round(w / sw.float()[:, None]), -8, 7).to(torch.int8)
        return agq.pack_w4(wq), sw

    # ---- decode: 224 distinct weight matrices
    layers = []
    for _ in range(synth.LLAMA7B_LAYERS):
        layers.append([(K, N) + make_packed(N, K) for (_, K, N) in synth.LLAMA7B_PROJ])
    weight_bytes = sum(p.numel() for layer in layers for (_, _, p, _) in layer)
    xs, es, ys = {}, {}, {}
    for M in DECODE_M:
        for K in (4096, 11008):
            x = torch.from_numpy(synth.make_activation(M, K, 4, seed=1)).to(dev)
            xs[(M, K)] = x
            es[(M, K)] = int(agq.calibrate_act_exp(x, 8).item())
    torch.cuda.synchronize()

    # One decode pass over a block: q, k and v read the same activation and run as
    # one agq_gemm_w4a8_multi call (one kernel launch), then o, then gate and up
    # as one call, then down: four launches for seven projections, each with its
    # own weights, scales and output.  --per-projection issues seven single calls.
    for M in DECODE_M:
        for name in ("q", "k", "v", "o", "down"):
            ys[(M, name)] = torch.empty((M, 4096), dtype=torch.float16, device=dev)
        for name in ("gate", "up"):
            ys[(M, name)] = torch.empty((M, 11008), dtype=torch.float16, device=dev)
    NAMES = ("q", "k", "v", "o", "gate", "up", "down")

    def single(M, layer, idx, bits=8):
        K, N, packed, sw = layer[idx]
        fn = agq.gemm_w4a8 if bits == 8 else agq.gemm_w4a4
        fn(xs[(M, K)], es[(M, K)] + (8 - bits), packed, sw, N, K, y=ys[(M, NAMES[idx])])

    def multi(M, layer, idxs, bits=8):
        K = layer[idxs[0]][0]
        projs = [(layer[i][2], layer[i][3], layer[i][1], ys[(M, NAMES[i])], None) for i in idxs]
        fn = agq.gemm_w4a8_multi if bits == 8 else agq.gemm_w4a4_multi
        fn(xs[(M, K)], es[(M, K)] + (8 - bits), projs, K)

    def decode_pass(M, bits=8):
        # the 4-bit activation grid takes the 8-bit exponent plus four: the same range in sixteen steps
        for layer in layers:
            if args.per_projection:
                for idx in range(7):
                    single(M, layer, idx, bits)
            else:
                multi(M, layer, (0, 1, 2), bits)
                single(M, layer, 3, bits)
                multi(M, layer, (4, 5), bits)
                single(M, layer, 6, bits)

    def decode_step():
        for M in DECODE_M:
            decode_pass(M)

    launches_per_pass = len(layers) * (7 if args.per_projection else 4)
    launches_per_step = len(DECODE_M) * launches_per_pass
    bytes_per_step = sum(algorithmic_bytes(M, K, N) for M in DECODE_M for layer in layers for (K, N, _, _) in layer)

    def timed(fn, warmup, steps, stats=None):
        """Captures `fn` (a launch-bound chain of kernels) into a HIP graph, replays it
        `warmup` times untimed and `steps` times between events on the replay stream.  Returns the
        milliseconds from the event before the first timed replay to the event after the last;
        stats (a dict), when given, also receives the median and the minimum over the replays."""
        fn()                                   # first call outside capture (lazy module load)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            fn()
        for _ in range(warmup):
            graph.replay()
        torch.cuda.synchronize()
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(steps + 1)]
        ev[0].record()
        for i in range(steps):
            graph.replay()
            ev[i + 1].record()
        torch.cuda.synchronize()
        if stats is not None:
            per = sorted(ev[i].elapsed_time(ev[i + 1]) for i in range(steps))
            stats["median_ms"], stats["min_ms"] = per[len(per) // 2], per[0]
        return ev[0].elapsed_time(ev[steps])

    step_stats = {}
    ms_total = timed(decode_step, args.warmup, args.steps, step_stats)
    ms_per_step = ms_total / args.steps
    gbs = bytes_per_step / (ms_per_step * 1e-3) / 1e9
    avg_launch_us = ms_per_step * 1e3 / launches_per_step

    # per-M breakdown (same buffers, timed separately)
    per_m = {}
    for M in DECODE_M:
        def one():
            decode_pass(M)
        reps = max(3, args.steps // 3)
        ms = timed(one, 1, reps) / reps
        by = sum(algorithmic_bytes(M, K, N) for layer in layers for (K, N, _, _) in layer)
        per_m["M%d" % M] = {"ms_per_sweep": round(ms, 4), "GB/s": round(by / (ms * 1e-3) / 1e9, 1),
                            "frac_hbm": round(by / (ms * 1e-3) / 1e9 / HBM_PEAK_GBS, 4)}

    # the same sweep with 4-bit activations (W4A4: Eq.2 with b = 4 in the prologue, same kernels and weights)
    per_m_a4 = {}
    for M in DECODE_M:
        def one4():
            decode_pass(M, 4)
        reps = max(3, args.steps // 3)
        ms = timed(one4, 1, reps) / reps
        by = sum(algorithmic_bytes(M, K, N) for layer in layers for (K, N, _, _) in layer)
        per_m_a4["M%d" % M] = {"ms_per_sweep": round(ms, 4), "GB/s": round(by / (ms * 1e-3) / 1e9, 1),
                               "frac_hbm": round(by / (ms * 1e-3) / 1e9 / HBM_PEAK_GBS, 4)}

    # the same sweep when the activation arrives as int8 codes (AGQ_X_Q: Eq.2 already applied once per tensor by
    # whatever produced it, outside the timed region): no quantizer, no LDS staging inside the GEMM
    per_m_xq = {}
    xq_codes = {key: agq.quantize_act(x, 8, es[key]) for key, x in xs.items()}

    def decode_pass_xq(M):
        for layer in layers:
            for idxs in ((0, 1, 2), (3,), (4, 5), (6,)):
                K = layer[idxs[0]][0]
                projs = [(layer[i][2], layer[i][3], layer[i][1], ys[(M, NAMES[i])], None) for i in idxs]
                agq.gemm_w4a8_multi(xq_codes[(M, K)], es[(M, K)], projs, K, x_kind=agq.AGQ_X_Q)

    for M in DECODE_M:
        reps = max(3, args.steps // 3)
        ms = timed(lambda: decode_pass_xq(M), 1, reps) / reps
        by = sum(algorithmic_bytes(M, K, N) - M * K for layer in layers for (K, N, _, _) in layer)   # int8 activation
        per_m_xq["M%d" % M] = {"ms_per_sweep": round(ms, 4), "GB/s": round(by / (ms * 1e-3) / 1e9, 1),
                               "frac_hbm": round(by / (ms * 1e-3) / 1e9 / HBM_PEAK_GBS, 4)}

    # one token row on the vector ALU (AGQ_X_F16_DOT: no LDS staging, no matrix core) against the library's own choice
    def decode_pass_dot(bits):
        fn = agq.gemm_w4a8_multi if bits == 8 else agq.gemm_w4a4_multi
        for layer in layers:
            for idxs in ((0, 1, 2), (3,), (4, 5), (6,)):
                K = layer[idxs[0]][0]
                projs = [(layer[i][2], layer[i][3], layer[i][1], ys[(1, NAMES[i])], None) for i in idxs]
                fn(xs[(1, K)], es[(1, K)] + (8 - bits), projs, K, x_kind=agq.AGQ_X_F16_DOT)

    dot_m1 = {}
    for bits in (8, 4):
        reps = max(3, args.steps // 3)
        ms = timed(lambda: decode_pass_dot(bits), 1, reps) / reps
        by = sum(algorithmic_bytes(1, K, N) for layer in layers for (K, N, _, _) in layer)
        dot_m1["w4a%d" % bits] = {"ms_per_sweep": round(ms, 4), "GB/s": round(by / (ms * 1e-3) / 1e9, 1),
                                  "frac_hbm": round(by / (ms * 1e-3) / 1e9 / HBM_PEAK_GBS, 4),
                                  "matrix_core_form_ms": (per_m if bits == 8 else per_m_a4)["M1"]["ms_per_sweep"]}

    result = {
        "metric": "W4A8 GEMM HBM GB/s, LLaMA-7B decode sweep (224 projections x M in {1,4,16})",
        "value": round(gbs, 1),
        "unit": "GB/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 4),
        "ms_per_step_median": round(step_stats["median_ms"], 4),
        "ms_per_step_min": round(step_stats["min_ms"], 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "int8 x int4 -> int32 (fp16 in/out)",
        "data": "synthetic",
        "config": {"workload": "llama7b_decode_w4a8: 32 blocks x 7 projections (4096->4096 x4, 4096->11008 x2, "
                               "11008->4096), M in {1,4,16}, 224 distinct packed weights",
                   "launches_per_step": launches_per_step, "weight_bytes": int(weight_bytes),
                   "algorithmic_bytes_per_step": int(bytes_per_step)},
        "roofline": {"bound": "hbm", "achieved": round(gbs, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(gbs / HBM_PEAK_GBS, 4), "traffic": measured_traffic("decode")[0],
                     "traffic_source": measured_traffic("decode")[1],
                     "kernel": "gemm_decode_kernel (one workgroup per 16-channel tile) and gemm_decode_slice_kernel (sixteen rows, several tiles per CU): "
                               "every launch of a step", "avg_launch_us": round(avg_launch_us, 3),
                     "algorithmic_bytes_per_launch": int(bytes_per_step / launches_per_step)},
        "decode_by_M": per_m,
        "decode_w4a4_by_M": per_m_a4,
        "decode_codes_in_by_M": per_m_xq,
        "decode_M1_vector_alu": dot_m1,
        "launch": "one HIP graph per step, replayed; per block: qkv (one multi call), o, gate+up (one multi call), down"
                  if not args.per_projection else "one HIP graph per step, replayed; seven single calls per block",
    }

    # ---- the same pass as ONE launch (agq_gemm_chain_*, M <= 4): every projection group is a stage of a persistent
    #      kernel; o reads the output of q (the attention output has that shape), gate/up the output of o, down the
    #      output of gate, the next block's q/k/v the output of down: a true dependency chain, as in a decode step.
    #      Exponents come from a calibration pass with single calls; scales are divided so that activations keep
    #      unit size along the 128 stages.  Reported beside the launch-per-group figures, not instead of them.
    if not args.no_chain:
        chain = {}
        unit_sw = [[(sw.float() / (0.02 * K ** 0.5)).to(torch.float16) for (K, N, _, sw) in layer] for layer in layers]
        for M in (1, 4):
            x0 = xs[(M, 4096)]
            stages, x = [], x0
            for li, L in enumerate(layers):
                def group(xin, idxs):
                    K = L[idxs[0]][0]
                    e = int(agq.calibrate_act_exp(xin, 8).item())
                    outs = agq.gemm_w4a8_multi(xin, e, [(L[i][2], unit_sw[li][i], L[i][1], None, None) for i in idxs], K)
                    st = dict(x=x0 if (li == 0 and idxs[0] == 0) else None, src_proj=0, bits=8, e=e, K=K,
                              projs=[(L[i][2], unit_sw[li][i], L[i][1], None, None) for i in idxs])
                    return st, outs
                st1, (q, _, _) = group(x, (0, 1, 2))
                st2, (o,) = group(q, (3,))
                st3, (g, _) = group(o, (4, 5))
                st4, (x,) = group(g, (6,))
                stages += [st1, st2, st3, st4]
            plan = agq.gemm_chain_prepare(stages, M)
            agq.gemm_chain_run(plan)
            torch.cuda.synchronize()
            same = bool(torch.equal(plan.ys[-1][0].view(torch.int16), x.view(torch.int16)))
            reps = max(5, args.steps)
            stc = {}
            ms = timed(lambda: agq.gemm_chain_run(plan), 2, reps, stc) / reps
            by = sum(algorithmic_bytes(M, K, N) for layer in layers for (K, N, _, _) in layer)
            chain["M%d" % M] = {"ms_per_pass": round(ms, 4), "ms_min": round(stc["min_ms"], 4), "us_per_stage": round(ms * 1e3 / len(stages), 2),
                                "GB/s": round(by / ms / 1e6, 1), "frac_hbm": round(by / ms / 1e6 / HBM_PEAK_GBS, 4),
                                "stages": len(stages), "status": agq.gemm_chain_status(plan),
                                "last_output_equals_single_calls": same}
            del plan, stages
        result["decode_chain"] = chain

    # ---- what one launch can reach on this device (the floor under the figures above): the same 128 launches
    #      of a pass as plain reads of buffers of the launches' sizes (q/k/v, o, gate/up, down of 32 blocks,
    #      3.2 GB in all, never cache-resident), and as empty kernels; replayed graphs, like the sweep itself
    if not args.no_probe:
        import ctypes
        probe = ctypes.CDLL(os.path.join(ROOT, "paper_2312_05693_amd", "libagq_probe.so"))
        probe.agq_probe_read.restype = ctypes.c_int
        probe.agq_probe_read.argtypes = [ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p, ctypes.c_void_p]
        probe.agq_probe_empty.restype = ctypes.c_int
        probe.agq_probe_empty.argtypes = [ctypes.c_void_p]
        sizes = [sum(layers[0][i][2].numel() for i in grp) for grp in ((0, 1, 2), (3,), (4, 5), (6,))]
        pool = torch.empty(sum(sizes) * len(layers), dtype=torch.uint8, device=dev).fill_(3)
        sink = torch.zeros(64, dtype=torch.int32, device=dev)
        stream_of = lambda: torch.cuda.current_stream().cuda_stream

        def read_pass():
            at = 0
            for _ in layers:
                for nb in sizes:
                    assert probe.agq_probe_read(pool.data_ptr() + at, nb, sink.data_ptr(), stream_of()) == 0
                    at += nb

        def empty_pass():
            for _ in range(4 * len(layers)):
                assert probe.agq_probe_empty(stream_of()) == 0

        n_l = 4 * len(layers)
        reps = max(5, args.steps)
        st_r, st_e = {}, {}
        ms_read = timed(read_pass, 2, reps, st_r) / reps
        ms_empty = timed(empty_pass, 2, reps, st_e) / reps
        per_size = {}
        for nb, name in zip(sizes, ("qkv", "o", "gate_up", "down")):
            def one_size():
                at = 0
                for _ in range(32):
                    assert probe.agq_probe_read(pool.data_ptr() + at, nb, sink.data_ptr(), stream_of()) == 0
                    at += nb
            us = timed(one_size, 2, reps) / reps / 32 * 1e3
            per_size[name] = {"MB": round(nb / 1e6, 1), "us": round(us, 2), "GB/s": round(nb / us / 1e3, 1)}
        read_gbs = pool.numel() / (ms_read * 1e-3) / 1e9
        result["probe"] = {
            "what": "the launches of one pass (32 blocks x 4) as plain reads of the same sizes, and as empty kernels, in replayed graphs",
            "read_GB/s": round(read_gbs, 1), "read_frac_of_peak": round(read_gbs / HBM_PEAK_GBS, 4),
            "read_us_per_launch": round(ms_read * 1e3 / n_l, 2), "read_us_per_launch_min": round(st_r["min_ms"] * 1e3 / n_l, 2),
            "empty_us_per_launch": round(ms_empty * 1e3 / n_l, 2), "empty_us_per_launch_min": round(st_e["min_ms"] * 1e3 / n_l, 2),
            "read_by_size": per_size,
            "note": "one launch per projection group cannot read faster than this: HBM requests start after the launch and "
                    "the last bytes arrive before the next launch begins"}
        result["roofline"]["frac_of_probe"] = round(gbs / read_gbs, 4)
        for k, v in per_m.items():
            v["frac_of_probe"] = round(v["GB/s"] / read_gbs, 4)
        del pool

    # ---- the small correctness configuration (one OPT-125M-sized layer, 128 tokens): launch-latency bound, time only
    x0 = torch.from_numpy(synth.make_activation(128, 768, 4, seed=0)).to(dev)
    p0w, s0w = make_packed(768, 768)
    e0 = int(agq.calibrate_act_exp(x0, 8).item())
    y0 = torch.empty((128, 768), dtype=torch.float16, device=dev)
    ws0 = torch.empty(max(agq.gemm_workspace_bytes(128, 768, 768), 16), dtype=torch.uint8, device=dev)
    def cfg0_calls():
        for _ in range(16):           # sixteen calls per replay: a replay of a single small node measures the replay
            agq.gemm_w4a8(x0, e0, p0w, s0w, 768, 768, y=y0, workspace=ws0)

    ms0 = timed(cfg0_calls, 2, 20) / 20 / 16
    result["config0_opt125m_w4a8"] = {"M": 128, "K": 768, "N": 768, "us": round(ms0 * 1e3, 2),
                                      "note": "151 Mop and 0.7 MB, latency bound: one launch of the weight-streaming "
                                              "kernel with eight row groups of 24 tile pairs (the tiled path would take two launches)"}

    # ---- prefill: one block's seven shapes at M = 2048, W4A8 and W4A4 (int8 MFMA bound)
    if not args.no_prefill:
        prefill = {}
        for name, fn, bits in (("w4a8", agq.gemm_w4a8, 8), ("w4a4", agq.gemm_w4a4, 4)):
            mfn = agq.gemm_w4a8_multi if bits == 8 else agq.gemm_w4a4_multi
            L = layers[0]
            xk = {K: torch.from_numpy(synth.make_activation(PREFILL_M, K, synth.n_outlier_channels(K), seed=2)).to(dev)
                  for K in (4096, 11008)}
            ek = {K: int(agq.calibrate_act_exp(xk[K], bits).item()) for K in xk}
            yk = [torch.empty((PREFILL_M, N), dtype=torch.float16, device=dev) for (_, _, N) in synth.LLAMA7B_PROJ]
            ws = torch.empty(agq.gemm_workspace_bytes(PREFILL_M, 4096, 11008), dtype=torch.uint8, device=dev)

            turn = [0]

            def block():
                # q/k/v share one quantize pre-pass, gate/up another: 4 pre-passes, 7 GEMMs.  Every call takes the
                # next block's weights (32 x 101 MB in rotation: nothing is left in a cache from the call before)
                L = layers[turn[0] % len(layers)]
                turn[0] += 1
                mfn(xk[4096], ek[4096], [(L[i][2], L[i][3], L[i][1], yk[i], None) for i in (0, 1, 2)], 4096, workspace=ws)
                fn(xk[4096], ek[4096], L[3][2], L[3][3], 4096, 4096, y=yk[3], workspace=ws)
                mfn(xk[4096], ek[4096], [(L[i][2], L[i][3], L[i][1], yk[i], None) for i in (4, 5)], 4096, workspace=ws)
                fn(xk[11008], ek[11008], L[6][2], L[6][3], 4096, 11008, y=yk[6], workspace=ws)

            def time_it(f, reps=30):
                for _ in range(10):          # the clocks settle only after a few milliseconds of load
                    f()
                torch.cuda.synchronize()
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record()
                for _ in range(reps):
                    f()
                b.record()
                torch.cuda.synchronize()
                return a.elapsed_time(b) / reps

            tot_ms = time_it(block)
            tot_ops = sum(2.0 * PREFILL_M * N * K for (_, K, N) in synth.LLAMA7B_PROJ)
            shapes = []
            for i in (0, 4, 6):       # one of each shape, single call with fp16 input (pre-pass included)
                pname, K, N = synth.LLAMA7B_PROJ[i]
                ms = time_it(lambda: fn(xk[K], ek[K], L[i][2], L[i][3], N, K, y=yk[i], workspace=ws))
                shapes.append({"proj": pname, "K": K, "N": N, "us": round(ms * 1e3, 2),
                               "TOP/s": round(2.0 * PREFILL_M * N * K / (ms * 1e-3) / 1e12, 1)})
            tops = tot_ops / (tot_ms * 1e-3) / 1e12
            prefill[name] = {"M": PREFILL_M, "ms_per_block": round(tot_ms, 4), "TOP/s": round(tops, 1),
                             "roofline": {"bound": "mfma", "achieved": round(tops, 1), "peak": INT8_PEAK_TOPS,
                                          "unit": "TOP/s", "frac": round(tops / INT8_PEAK_TOPS, 4),
                                          "traffic": measured_traffic("tiled")[0], "traffic_source": measured_traffic("tiled")[1],
                                          "kernel": "gemm_tiled_kernel",
                                          "note": "fp16 input: time includes the 4 quantize/layout pre-passes of a block"},
                             "single_calls": shapes}
        # Between the two regimes (W4A8, fp16 input, single calls over eight distinct weight matrices per shape in a
        # replayed graph): row groups of the weight-streaming kernel, then the tiled kernel with K split over
        # workgroups while it has few tiles
        by_m = []
        for i in (() if args.no_by_m else (0, 4, 6)):
            pname, K, N = synth.LLAMA7B_PROJ[i]
            row = {"proj": pname, "K": K, "N": N}
            e8 = int(agq.calibrate_act_exp(xk[K], 8).item())
            for M in (32, 64, 128, 256, 512, 1024):
                xm = xk[K][:M].contiguous()
                ym = torch.empty((M, N), dtype=torch.float16, device=dev)
                wsm = torch.empty(max(16, agq.gemm_workspace_bytes(M, N, K)), dtype=torch.uint8, device=dev)

                def calls():
                    for layer in layers[:8]:
                        agq.gemm_w4a8(xm, e8, layer[i][2], layer[i][3], N, K, y=ym, workspace=wsm)

                us = timed(calls, 3, 10) / 10 / 8 * 1e3
                row["M%d" % M] = {"us": round(us, 2), "TOP/s": round(2.0 * M * N * K / us / 1e6, 1)}
            by_m.append(row)
        if by_m:
            prefill["w4a8_by_M"] = by_m
        # The same GEMM launch (4096 -> 11008 at M = 2048, W4A8, codes handed over: the kernel alone) on random
        # operands and on all-zero operands: identical instructions and bytes, different switching activity
        pname, K, N = synth.LLAMA7B_PROJ[4]
        ent = {}
        for label in ("random", "zero"):
            if label == "random":
                xe, pe = xk[K], layers[0][4][2]
            else:
                xe = torch.zeros((PREFILL_M, K), dtype=torch.float16, device=dev)
                pe = agq.pack_w4(torch.zeros((N, K), dtype=torch.int8, device=dev))
            e8 = int(agq.calibrate_act_exp(xk[K], 8).item())
            xq = agq.quantize_act(xe, 8, e8)
            ye = torch.empty((PREFILL_M, N), dtype=torch.float16, device=dev)
            wse = torch.empty(agq.gemm_workspace_bytes(PREFILL_M, N, K), dtype=torch.uint8, device=dev)
            ms = time_it(lambda: agq.gemm_w4a8(xq, e8, pe, layers[0][4][3], N, K, x_kind=agq.AGQ_X_Q, y=ye, workspace=wse), reps=50)
            ent[label] = {"us": round(ms * 1e3, 2), "TOP/s": round(2.0 * PREFILL_M * N * K / (ms * 1e-3) / 1e12, 1)}
        ent["note"] = "same launch, same instruction stream and bytes; only the operand values differ"
        prefill["operand_values_w4a8_4096_to_11008"] = ent
        # What the matrix cores sustain on this device for the kernel's instruction (16 x 16 x 64 int8 MFMA, two
        # wavefronts per SIMD, eight independent accumulators, no memory traffic): with all-zero operands, with
        # operand values taken from the workload (weights as the kernels feed them, 16 w, and the activation's
        # 8-bit codes) and with uniformly random bytes.  The instruction stream is the same in all three; the
        # 32 x 32 x 32 form beside it.
        if not args.no_probe:
            import ctypes
            probe = ctypes.CDLL(os.path.join(ROOT, "paper_2312_05693_amd", "libagq_probe.so"))
            probe.agq_probe_mfma_i8.restype = ctypes.c_int
            probe.agq_probe_mfma_i8.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_int,
                                                ctypes.c_void_p, ctypes.c_void_p]
            gen_p = torch.Generator(device=dev)
            gen_p.manual_seed(11)
            nb_p = 16384                                  # operand bytes per side: four registers sets per lane
            w16 = (torch.randint(-8, 8, (nb_p,), generator=gen_p, device=dev, dtype=torch.int8) * 16).contiguous()
            codes = agq.quantize_act(xk[4096][:4].contiguous(), 8, ek[4096]).reshape(-1)[:nb_p].contiguous()
            rnd = torch.randint(-128, 128, (2 * nb_p,), generator=gen_p, device=dev, dtype=torch.int8)
            zero = torch.zeros(nb_p, dtype=torch.int8, device=dev)
            sink_p = torch.zeros(64, dtype=torch.int32, device=dev)
            wgs, reps_p = 512, 20000                     # two workgroups of four wavefronts per CU
            ops = 8.0 * 32 ** 3 * reps_p * wgs * 4
            mp = {}
            r0, r1 = rnd[:nb_p].contiguous(), rnd[nb_p:].contiguous()
            for label, pa, pb, wide in (("zero_operands", zero, zero, 0), ("workload_operands", w16, codes, 0),
                                        ("uniform_random_bytes", r0, r1, 0), ("zero_operands_32x32x32", zero, zero, 1),
                                        ("workload_operands_32x32x32", w16, codes, 1), ("uniform_random_bytes_32x32x32", r0, r1, 1)):
                launch = lambda: probe.agq_probe_mfma_i8(pa.data_ptr(), pb.data_ptr(), wgs, reps_p, wide, sink_p.data_ptr(),
                                                         torch.cuda.current_stream().cuda_stream)
                assert launch() == 0
                torch.cuda.synchronize()
                best = 1e9
                for _ in range(3):
                    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                    e0.record()
                    assert launch() == 0
                    e1.record()
                    torch.cuda.synchronize()
                    best = min(best, e0.elapsed_time(e1))
                mp[label + "_TOP/s"] = round(ops / (best * 1e-3) / 1e12, 1)
            mp["what"] = ("the tiled kernel's matrix instruction alone (no loads, no LDS; every MFMA with other operand "
                          "registers than the one before), 512 workgroups of four wavefronts, ~2 ms each: the rate the "
                          "matrix cores sustain depends on the operand values")
            prefill["mfma_probe"] = mp
            for name in ("w4a8", "w4a4"):
                prefill[name]["roofline"]["frac_of_probe"] = round(prefill[name]["TOP/s"] / mp["workload_operands_TOP/s"], 4)
        result["prefill"] = prefill

    # ---- TRIP (Section 4.3 / 4.4): the same three shapes with per-channel factors found by Eq.8 on a
    #      2048-token activation with 1 % outlier channels; decode launches (single calls, 12 distinct
    #      blobs per shape in rotation) and the M = 2048 GEMM, beside the plain layer on the same inputs
    if not args.no_trip:
        trip = {"workload": "llama7b shapes, W4A8 with TRIP factors (K = 4 refinements), fp16 input", "shapes": []}
        kmax, copies = 4, 12
        for (pname, K, N) in (synth.LLAMA7B_PROJ[0], synth.LLAMA7B_PROJ[4], synth.LLAMA7B_PROJ[6]):
            xcal = torch.from_numpy(synth.make_activation(PREFILL_M, K, synth.n_outlier_channels(K), seed=2)).to(dev)
            e_layer = int(agq.calibrate_act_exp(xcal, 8).item())
            alpha = agq.trip_search(xcal, 8, e_layer - kmax, kmax).cpu().numpy()
            blobs_t, blobs_p = [], []
            for _ in range(copies):
                w = torch.randn((N, K), generator=gen, device=dev, dtype=torch.float32) * 0.02
                sw = (w.abs().amax(dim=1) / 7.0).to(torch.float16)
                wq = torch.clamp(torch.round(w / sw.float()[:, None]), -8, 7).to(torch.int8)
                bt, n_extra = agq.pack_w4_trip(wq, alpha)
                blobs_t.append((bt, sw))
                blobs_p.append((agq.pack_w4(wq), sw))
                del w, wq
            entry = {"proj": pname, "K": K, "N": N, "channels_with_factor": int((alpha > 0).sum()),
                     "extra_chunks": n_extra, "decode": {}}
            for M in DECODE_M:
                xm = xcal[:M].contiguous()
                ym = torch.empty((M, N), dtype=torch.float16, device=dev)

                def run_t():
                    for (b, sw) in blobs_t:
                        agq.gemm_trip(xm, 8, e_layer - kmax, b, n_extra, sw, N, K, y=ym)

                def run_p():
                    for (b, sw) in blobs_p:
                        agq.gemm_w4a8(xm, e_layer, b, sw, N, K, y=ym)

                us_t = timed(run_t, 2, 10) / 10 / copies * 1e3
                us_p = timed(run_p, 2, 10) / 10 / copies * 1e3
                by = algorithmic_bytes(M, K, N) + n_extra * 64 * N + n_extra * 128 * (4 + 2 * M)
                entry["decode"]["M%d" % M] = {"us": round(us_t, 2), "us_plain": round(us_p, 2),
                                               "GB/s": round(by / us_t / 1e3, 1),
                                               "frac_hbm": round(by / us_t / 1e3 / HBM_PEAK_GBS, 4)}
            ws_t = torch.empty(agq.lib().agq_gemm_trip_workspace_bytes(PREFILL_M, N, K, n_extra), dtype=torch.uint8, device=dev)
            yp = torch.empty((PREFILL_M, N), dtype=torch.float16, device=dev)

            def pre_t():
                agq.gemm_trip(xcal, 8, e_layer - kmax, blobs_t[0][0], n_extra, blobs_t[0][1], N, K, y=yp, workspace=ws_t)

            def pre_p():
                agq.gemm_w4a8(xcal, e_layer, blobs_p[0][0], blobs_p[0][1], N, K, y=yp, workspace=ws_t)

            def time_eager(f, reps=30):
                for _ in range(10):
                    f()
                torch.cuda.synchronize()
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record()
                for _ in range(reps):
                    f()
                b.record()
                torch.cuda.synchronize()
                return a.elapsed_time(b) / reps * 1e3

            us_t, us_p = time_eager(pre_t), time_eager(pre_p)
            ops = 2.0 * PREFILL_M * N * (K + 128 * n_extra)
            entry["prefill_M%d" % PREFILL_M] = {"us": round(us_t, 1), "us_plain": round(us_p, 1),
                                                "TOP/s": round(ops / us_t / 1e6, 1),
                                                "frac_mfma": round(ops / us_t / 1e6 / INT8_PEAK_TOPS, 4)}
            trip["shapes"].append(entry)
            del blobs_t, blobs_p, xcal
        result["trip"] = trip

    def time_plain(f, reps=20):
        """ms per call, eager launches on the current stream (events recorded on that stream)"""
        for _ in range(10):
            f()
        torch.cuda.synchronize()
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(reps):
            f()
        b.record()
        torch.cuda.synchronize()
        return a.elapsed_time(b) / reps

    # ---- attention side path at LLaMA-13B size: log2-quantized softmax x V with the start-token score,
    #      then Eq.4 pruning to half the tokens (HBM bound: the probabilities are read once)
    if not args.no_attention:
        H, S, D = 40, 2048, 128
        g2 = torch.Generator(device=dev)
        g2.manual_seed(4)
        qh = torch.randn(H, S, D, generator=g2, device=dev)
        kh = torch.randn(H, S, D, generator=g2, device=dev)
        logits = qh @ kh.transpose(1, 2) / D ** 0.5
        logits[:, :, 0] += 4.0                                           # the start-token stripe of Section 4.3
        causal = torch.tril(torch.ones(S, S, dtype=torch.bool, device=dev))
        p0 = torch.softmax(logits.masked_fill(~causal, float("-inf")), dim=-1).to(torch.float16).contiguous()
        del qh, kh, logits, causal
        probs = [p0, p0.clone(), p0.clone()]                              # 1 GB in rotation: no cache reuse between calls
        vq = torch.randint(-127, 128, (H, S, D), generator=g2, device=dev, dtype=torch.int8)
        turn = [0]

        def attn():
            turn[0] += 1
            return agq.log2_quant_softmax(probs[turn[0] % 3], vq, -5)

        us_attn = time_plain(attn) * 1e3
        o_a, _, score_a = attn()
        us_prune = time_plain(lambda: agq.prune_tokens(score_a, S // 2, o_a)) * 1e3
        # the two W4A8 projections that follow on the 1024 surviving tokens (int8 MFMA bound)
        hid, ffn, keep = H * D, 13824, S // 2
        _, xp = agq.prune_tokens(score_a, keep, o_a)
        tail_w = [make_packed(hid, hid), make_packed(ffn, hid)]
        y1 = torch.empty((keep, hid), dtype=torch.float16, device=dev)
        y2 = torch.empty((keep, ffn), dtype=torch.float16, device=dev)
        e1 = int(agq.calibrate_act_exp(xp, 8).item())
        ws_t = torch.empty(agq.gemm_workspace_bytes(keep, ffn, hid), dtype=torch.uint8, device=dev)
        agq.gemm_w4a8(xp, e1, tail_w[0][0], tail_w[0][1], hid, hid, y=y1, workspace=ws_t)
        e2 = int(agq.calibrate_act_exp(y1, 8).item())

        def tail():
            agq.gemm_w4a8(xp, e1, tail_w[0][0], tail_w[0][1], hid, hid, y=y1, workspace=ws_t)
            agq.gemm_w4a8(y1, e2, tail_w[1][0], tail_w[1][1], ffn, hid, y=y2, workspace=ws_t)

        us_tail = time_plain(tail, reps=20) * 1e3
        ops_tail = 2.0 * keep * hid * (hid + ffn)
        by_attn = H * S * (S + 1) // 2 * 2 + H * S * D + S * H * D * 2       # causal half of P, V, O
        by_prune = 4 * S + 2 * (S // 2) * H * D * 2
        result["attention"] = {
            "workload": "llama13b attention block: H=40, S=2048, D=128, causal, qmax=15, prune to 1024 tokens",
            "log2_softmax_v": {"us": round(us_attn, 1), "GB/s": round(by_attn / us_attn / 1e3, 1),
                               "roofline": {"bound": "hbm", "achieved": round(by_attn / us_attn / 1e3, 1),
                                            "peak": HBM_PEAK_GBS, "unit": "GB/s",
                                            "frac": round(by_attn / us_attn / 1e3 / HBM_PEAK_GBS, 4),
                                            "traffic": measured_traffic("attn")[0], "traffic_source": measured_traffic("attn")[1],
                                            "kernel": "log2_attn_kernel"}},
            "prune_tokens": {"us": round(us_prune, 1), "GB/s": round(by_prune / us_prune / 1e3, 1)},
            "tail_gemms_w4a8": {"M": keep, "shapes": "5120->5120, 5120->13824", "us": round(us_tail, 1),
                                "TOP/s": round(ops_tail / us_tail / 1e6, 1),
                                "frac_mfma": round(ops_tail / us_tail / 1e6 / INT8_PEAK_TOPS, 4)}}
        del probs, p0

        # the same block from quantized Q and K in one kernel (no probabilities in memory): int8 Q K^T,
        # softmax statistics, Eq.3 codes and the product with V
        mk8 = lambda: torch.clamp(torch.round(torch.randn(H, S, D, generator=g2, device=dev) * 32), -127, 127).to(torch.int8)
        q8, k8 = mk8(), mk8()
        us_qk = time_plain(lambda: agq.qk_log2_softmax(q8, k8, vq, -5, -5, -5)) * 1e3
        pairs = H * S * (S + 1) // 2
        ops_i8, ops_f16 = 2.0 * pairs * D, 2.0 * pairs * D            # one Q K^T (int8) and one P V (fp16), algorithmic
        ideal_us = ops_i8 / (INT8_PEAK_TOPS * 1e6) + ops_f16 / (F16_PEAK_TFLOPS * 1e6)
        result["attention"]["qk_log2_softmax_v"] = {
            "us": round(us_qk, 1), "inputs": "int8 Q, K, V [40, 2048, 128]",
            "roofline": {"bound": "mfma", "achieved": round((ops_i8 + ops_f16) / us_qk / 1e6, 1),
                         "peak": round((ops_i8 + ops_f16) / ideal_us / 1e6, 1), "unit": "TOP/s",
                         "frac": round(ideal_us / us_qk, 4), "traffic": None, "kernel": "qk_log2_attn_kernel",
                         "note": "algorithmic ops: one int8 Q K^T and one fp16 P V over the causal pairs; peak = "
                                 "those ops at 5.0 POP/s and 2.5 PFLOP/s; the kernel computes Q K^T twice (two passes)"}}

    # ---- one whole block of the pipeline (Section 4.2, Figure 3): RMSNorm, q/k/v, rotary embedding + Eq.2,
    #      attention from int8 Q and K, pruning (Section 4.3), 4-bit projection after attention, residual,
    #      RMSNorm, gate/up, SwiGLU, down, residual; 2048 tokens in, all of them or half of them out
    if not args.no_block:
        def unit_packed(N, K):
            w = torch.randn((N, K), generator=gen, device=dev, dtype=torch.float32)
            sw = w.abs().amax(dim=1) / 7.0
            wq = torch.clamp(torch.round(w / sw[:, None]), -8, 7).to(torch.int8)
            return agq.pack_w4(wq), (sw / K ** 0.5).to(torch.float16)      # unit-scale residual stream

        blocks = []
        for (model, d, H, F) in (("llama13b", 5120, 40, 13824), ("llama7b", 4096, 32, 11008)):
            S = PREFILL_M
            wts = {"g_attn": torch.ones(d, dtype=torch.float16, device=dev), "g_mlp": torch.ones(d, dtype=torch.float16, device=dev)}
            for n, (N, K) in dict(q=(d, d), k=(d, d), v=(d, d), o=(d, d), gate=(F, d), up=(F, d), down=(d, F)).items():
                wts["w_" + n], wts["s_" + n] = unit_packed(N, K)
            xb = torch.from_numpy(synth.make_activation(S, d, synth.n_outlier_channels(d), seed=5)).to(dev)
            posb = torch.arange(S, dtype=torch.int32, device=dev)
            cs, sn = synth.rope_tables(S, d // H)
            cs, sn = torch.from_numpy(cs).to(dev), torch.from_numpy(sn).to(dev)
            entry = {"model": model, "d": d, "H": H, "F": F, "S": S}
            for keep in (S, S // 2):
                blk = agq.make_block(d, H, F, wts, qmax=15, bits_attn_out=4, rms_eps=1e-5)
                xo, po, wsb, _ = agq.block_forward(blk, xb, posb, cs, sn, n_keep=keep, calibrate=True)
                # the call enqueues kernels only: captured once, replayed (as the decode sweep is)
                ms = timed(lambda: agq.block_forward(blk, xb, posb, cs, sn, n_keep=keep, workspace=wsb, out=(xo, po)), 10, 20) / 20
                pairs = H * S * (S + 1) // 2
                ops = 2.0 * S * d * 3 * d + 4.0 * pairs * (d // H) + 2.0 * keep * d * d + 6.0 * keep * d * F
                entry["keep_%d" % keep] = {"ms": round(ms, 4), "tokens_in/s": round(S / ms * 1e3, 0),
                                           "products_TOP/s": round(ops / ms / 1e9, 1), "exps": agq.block_exps(blk)}
                del wsb
            if model == "llama13b":
                # TRIP (Section 4.3) at the two normalised activations (q/k/v and gate/up inputs, where the outlier
                # channels sit): factors by Eq.8 on the tensors of the calibration pass, base step per Eq.6
                S_, keep = S, S
                blk = agq.make_block(d, H, F, wts, qmax=15, bits_attn_out=4, rms_eps=1e-5)
                xo, po, wsb, Lb = agq.block_forward(blk, xb, posb, cs, sn, n_keep=keep, calibrate=True)
                exps_t, trip_n, wts_t, kmax = agq.block_exps(blk), {}, dict(wts), 4
                for site, src, names in (("attn_in", "h1", ("q", "k", "v")), ("mlp_in", "h2", ("gate", "up"))):
                    t_site = agq.block_tensor(blk, Lb, wsb, src, S_, keep)
                    exps_t["e_" + site] -= kmax
                    alpha = agq.trip_search(t_site, 8, exps_t["e_" + site], kmax).cpu().numpy()
                    for n in names:
                        N, K = (d, d) if site == "attn_in" else (F, d)
                        wq_n = agq.unpack_w4(wts["w_" + n], N, K)
                        wts_t["w_" + n], trip_n[site] = agq.pack_w4_trip(wq_n, alpha)
                        del wq_n
                    entry["trip_" + site] = {"channels_with_factor": int((alpha > 0).sum()), "extra_chunks": trip_n[site]}
                del wsb
                blk_t = agq.make_block(d, H, F, wts_t, qmax=15, bits_attn_out=4, rms_eps=1e-5, exps=exps_t, trip=trip_n)
                xo, po, wsb, _ = agq.block_forward(blk_t, xb, posb, cs, sn, n_keep=keep)
                ms = timed(lambda: agq.block_forward(blk_t, xb, posb, cs, sn, n_keep=keep, workspace=wsb, out=(xo, po)), 10, 20) / 20
                entry["keep_%d_trip" % keep] = {"ms": round(ms, 4), "tokens_in/s": round(S / ms * 1e3, 0)}
                del wsb, wts_t
            blocks.append(entry)
            del wts, xb
        # a stack of four LLaMA-13B-shaped blocks (distinct weights) in one call: without pruning, and with Eq.9's
        # cascade (beta = 0.5 over two stages, applied in blocks 1 and 3)
        d, H, F, S, nb = 5120, 40, 13824, PREFILL_M, 4
        xb = torch.from_numpy(synth.make_activation(S, d, synth.n_outlier_channels(d), seed=5)).to(dev)
        posb = torch.arange(S, dtype=torch.int32, device=dev)
        cs, sn = synth.rope_tables(S, d // H)
        cs, sn = torch.from_numpy(cs).to(dev), torch.from_numpy(sn).to(dev)
        stack_w = []
        for _ in range(nb):
            wts = {"g_attn": torch.ones(d, dtype=torch.float16, device=dev), "g_mlp": torch.ones(d, dtype=torch.float16, device=dev)}
            for n, (N, K) in dict(q=(d, d), k=(d, d), v=(d, d), o=(d, d), gate=(F, d), up=(F, d), down=(d, F)).items():
                wts["w_" + n], wts["s_" + n] = unit_packed(N, K)
            stack_w.append(wts)
        stages = agq.cascade_keep(S, 0.5, 2)
        stack = {"model": "llama13b", "blocks": nb, "S": S}
        for name, keep in (("dense", [S] * nb), ("cascade", [S, stages[0], stages[0], stages[1]])):
            blks, xg, pg = [], xb, posb
            for l in range(nb):                   # calibrate every block on the tokens it receives
                blk = agq.make_block(d, H, F, stack_w[l], qmax=15, bits_attn_out=4, rms_eps=1e-5)
                xg, pg, _, _ = agq.block_forward(blk, xg, pg, cs, sn, n_keep=keep[l], calibrate=True)
                blks.append(blk)
            xo, po, wss = agq.stack_forward(blks, keep, xb, posb, cs, sn)
            ms = timed(lambda: agq.stack_forward(blks, keep, xb, posb, cs, sn, workspace=wss, out=(xo, po)), 5, 10) / 10
            stack[name] = {"keep": keep, "ms": round(ms, 4), "tokens_in/s": round(S / ms * 1e3, 0)}
            del wss, blks
        del stack_w, xb
        result["block_stack"] = stack
        result["block"] = {"workload": "one LLaMA block of the quantized pipeline, 2048 tokens, W4A8 with 4-bit activations "
                                       "after attention, without pruning and pruning to half after attention",
                           "blocks": blocks}

    # ---- CPU baseline: the oracle as it stands, on a bounded sample of the decode workload
    if not args.no_cpu_baseline:
        from oracle import build as oracle_build
        oracle_build.build()
        from oracle import agq_oracle as oracle
        threads = oracle.c_max_threads()
        cpu_layer = [(K, N) + synth.make_weight_q4(N, K, seed=100 + i) for i, (_, K, N) in enumerate(synth.LLAMA7B_PROJ)]
        cpu_x = {(M, K): synth.make_activation(M, K, 4, seed=1) for M in DECODE_M for K in (4096, 11008)}

        def cpu_rate(nthreads, budget_s):
            t_start = time.perf_counter()
            done_bytes, passes = 0, 0
            while time.perf_counter() - t_start < budget_s and passes < 400:
                for M in DECODE_M:
                    for (K, N, wq, sw) in cpu_layer:
                        x = cpu_x[(M, K)]
                        e = es[(M, K)]
                        q = oracle.quantize_act(x, 8, e, 0).astype(np.int8)
                        acc = oracle.gemm_int_c(q, wq, threads=nthreads)
                        oracle.dequant_out(acc, e, sw)
                        done_bytes += algorithmic_bytes(M, K, N)
                passes += 1
            cpu_s = time.perf_counter() - t_start
            return done_bytes / cpu_s / 1e9, passes, cpu_s

        rate_all, passes, cpu_s = cpu_rate(threads, 10.0)
        rate_one, passes1, cpu_s1 = cpu_rate(1, 8.0)
        result["cpu_baseline"] = {"value": round(rate_all, 3), "unit": "GB/s", "cores": threads,
                                  "kind": "oracle",
                                  "sample": "%d pass(es) over one block's 7 projections x M in {1,4,16} "
                                            "(numpy quantizer + plain C int8 loops + numpy dequant), %.1f s" % (passes, cpu_s),
                                  "value_1_thread": round(rate_one, 3),
                                  "sample_1_thread": "%d pass(es) of the same, %.1f s" % (passes1, cpu_s1)}

    print(json.dumps(result))


if __name__ == "__main__":
    main()
