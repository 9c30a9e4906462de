#!/usr/bin/env python3
"""Benchmark of libkata's causal KATA-M1 forward on one MI355X.

A step is one pass of the chunked-state forward (span state -> associative scan
-> fused intra-span attention + prefix readout + normalisation) over one batch
of the long-context workload: B=1, H=16, T=131072, d=dv=64, chunk C=64, bf16
q/k/v with fp32 accumulation, inputs resident in HBM.  Prints ONE JSON line.

Per-kernel durations are taken live with HIP events recorded on the launch
stream between the three kernels (kata_fwd_chunked_timed).  The decode
workload (B=256, H=16, 1024-token prefix, 128 steps) is measured in the same
run and reported under "decode"; KATA-M2 under "m2"; the quadratic form
against the chunked one under "quadratic_vs_chunked"; causal linear attention
with the linear feature maps (the paper's associative-scan shape, B=1, H=16,
d=64, C=128) under "linear_features"; the training step (forward + chunked
backward) at B=8, H=16, d=64 under "backward".  The CPU oracle is timed on a bounded
sample of rows of the same workload and reported under "cpu_baseline".
"""
from __future__ import annotations

import argparse
import ctypes
import hashlib
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "KATA causal fwd tokens/s at T=131k,d=64 (1 GPU); % bf16 MFMA peak"
PEAK_BF16_TFLOPS = 2500.0      # MI355X dense bf16 MFMA
PEAK_HBM_GBS = 8000.0          # MI355X HBM3E
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "traffic_counters.json")


def _hip():
    L = ctypes.CDLL("libamdhip64.so")
    vp = ctypes.c_void_p
    L.hipEventCreate.argtypes = [ctypes.POINTER(vp)]
    L.hipEventRecord.argtypes = [vp, vp]
    L.hipEventSynchronize.argtypes = [vp]
    L.hipEventElapsedTime.argtypes = [ctypes.POINTER(ctypes.c_float), vp, vp]
    L.hipEventDestroy.argtypes = [vp]
    return L


class Events:
    def __init__(self, hip, n):
        self.hip = hip
        self.ev = (ctypes.c_void_p * n)()
        for i in range(n):
            h = ctypes.c_void_p()
            assert hip.hipEventCreate(ctypes.byref(h)) == 0
            self.ev[i] = h

    def elapsed(self, i, j):
        ms = ctypes.c_float()
        assert self.hip.hipEventElapsedTime(ctypes.byref(ms), self.ev[i], self.ev[j]) == 0
        return ms.value

    def record(self, i, stream):
        """Record event i on `stream` (a torch stream)."""
        self.hip.hipEventRecord.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
        assert self.hip.hipEventRecord(self.ev[i], ctypes.c_void_p(stream.cuda_stream)) == 0

    def block(self, i):
        """Pointer to 4 consecutive events starting at index i."""
        return ctypes.c_void_p(ctypes.addressof(self.ev) + i * ctypes.sizeof(ctypes.c_void_p))

    def close(self):
        for e in self.ev:
            self.hip.hipEventDestroy(e)


M1_SOURCES = ("kata_mfma.hip", "kata_scan.hpp", "kata_common.hpp")
LIN_SOURCES = ("kata_linear.hip", "kata_scan.hpp", "kata_common.hpp")


def source_sha(files=M1_SOURCES):
    h = hashlib.sha256()
    for f in files:
        with open(os.path.join(ROOT, "paper_2607_17419_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def upload(payload, dtype, dev):
    import numpy as np
    import torch
    if dtype == "bf16":
        return torch.from_numpy(np.ascontiguousarray(payload).view(np.int16)).to(dev).view(torch.bfloat16)
    return torch.from_numpy(np.ascontiguousarray(payload)).to(dev)


def algorithmic(w, L, g=1):
    """Algorithmic work per kernel (packed n = d(d+1)/2 features; with g
    feature blocks of KATA-Mg, n = g*m(m+1)/2 with m = d/g).

    per head-token:  state   2*n*dv + n          (S += phi(k) v^T, z += phi(k))
                     output  2*n*dv + 2*n + (C+1)*(d+dv)
                             (phi(q)^T S and phi(q)^T z readouts, causal
                              intra-chunk QK^T and PV at chunk size C)
    The state term counts every key but those of the last chunk (its state
    enters no exclusive prefix) and the readout term every query but those of
    the first chunk (its prefix is zero).
    scan: one bf16 read of every span state but the last (n*(dv+1) values;
          the last span's state enters no exclusive prefix) and one bf16
          write of every span's exclusive prefix, per head.
    """
    m = w.d // g
    n = g * (m * (m + 1) // 2)
    bh = w.B * w.H
    ht = bh * w.T
    NS = (w.T + L - 1) // L
    NC = (w.T + w.C - 1) // w.C
    state = (2 * n * w.dv + n) * bh * (NC - 1) * w.C
    output = ((2 * n * w.dv + 2 * n) * bh * (w.T - min(w.C, w.T))
              + (w.C + 1) * (w.d + w.dv) * ht)
    scan_bytes = (2 * NS - 1) * w.B * w.H * n * (w.dv + 1) * 2
    return dict(n=n, state_flop=state, output_flop=output, scan_bytes=scan_bytes,
                total_flop=state + output)


def bench_fwd(kata, dev, hip, w, steps, warmup, span=0, inp=None):
    """Chunked forward of workload `w` (inputs resident on the device): wall
    time per step over `steps` calls after `warmup`, and per-stage times from
    the HIP events the library records on the launch stream between its three
    kernels (span / chunk state, associative scan, output)."""
    import torch
    if inp is None:
        import workloads
        inp = workloads.make_inputs(w)
    q = upload(inp["q_dev"], w.dtype, dev)
    k = upload(inp["k_dev"], w.dtype, dev)
    v = upload(inp["v_dev"], w.dtype, dev)
    code = kata.KATA_BF16 if w.dtype == "bf16" else kata.KATA_F32
    span = span or kata.default_span(w.B, w.H, w.T, w.d, w.dv, w.C, code)
    L = min(span * w.C, -(-w.T // w.C) * w.C)
    out = torch.empty((w.B, w.H, w.T, w.dv), dtype=torch.float32, device=dev)
    ws = torch.empty(max(256, kata.workspace_bytes(w.B, w.H, w.T, w.d, w.dv, w.C, code, span)),
                     dtype=torch.uint8, device=dev)
    ev = Events(hip, 4 * max(steps, warmup))
    for i in range(warmup):
        kata.fwd_chunked_timed(q, k, v, w.C, ev.block(4 * i), span_chunks=span, out=out,
                               workspace=ws)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(steps):
        kata.fwd_chunked_timed(q, k, v, w.C, ev.block(4 * i), span_chunks=span, out=out,
                               workspace=ws)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    names = ("span_state", "scan", "span_output")
    stage = {nm: sum(ev.elapsed(4 * i + j, 4 * i + j + 1) for i in range(steps)) / steps
             for j, nm in enumerate(names)}
    ev.close()
    ms = 1e3 * elapsed / steps
    res = {"ms": ms, "stage": stage, "span": span, "L": L, "code": code}
    return res, (q, k, v)


def fwd_row(w, r):
    """Summary of one forward workload: tokens/s, stage times, and on the bf16
    MFMA path the MFMA fractions of the state and output kernels (algorithmic
    flops) and the scan's HBM rate (algorithmic bytes)."""
    alg = algorithmic(w, r["L"])
    st = r["stage"]
    row = {"workload": f"{w.name}: {w.note}", "tokens_per_s": w.B * w.T / (r["ms"] * 1e-3),
           "ms_per_step": round(r["ms"], 4), "kernel_ms": round(sum(st.values()), 4),
           "span_chunks": r["span"], "stages_ms": {nm: round(t, 4) for nm, t in st.items()}}
    if w.dtype == "bf16":
        def mf(flop, t_ms):
            tf = flop / (t_ms * 1e-3) / 1e12
            return {"bound": "mfma", "achieved": round(tf, 2), "peak": PEAK_BF16_TFLOPS,
                    "unit": "TFLOP/s", "frac": round(tf / PEAK_BF16_TFLOPS, 4)}
        gbs = alg["scan_bytes"] / (st["scan"] * 1e-3) / 1e9
        row["stage_roofline"] = {
            "span_state": mf(alg["state_flop"], st["span_state"]),
            "span_output": mf(alg["output_flop"], st["span_output"]),
            "scan": {"bound": "hbm", "achieved": round(gbs, 1), "peak": PEAK_HBM_GBS,
                     "unit": "GB/s", "frac": round(gbs / PEAK_HBM_GBS, 4)}}
        row["mfma_frac_end_to_end"] = round(
            alg["total_flop"] / (r["ms"] * 1e-3) / 1e12 / PEAK_BF16_TFLOPS, 4)
        row["algorithmic_gflop_per_step"] = round(alg["total_flop"] / 1e9, 2)
    else:
        row["note"] = ("fp32 inputs of this length run in the quadratic form on the fp32 matrix cores; "
                       "latency-bound at this size, reported as time per call")
    return row


def bench_configs(kata, dev, hip, names=("tiny_f32", "mid_bf16", "recall_bf16"), steps=20,
                  warmup=5):
    """The other forward workloads, each in the library's default launch
    configuration (default span), on their seeded inputs."""
    import torch
    import workloads
    out = {}
    for nm in names:
        w = workloads.WORKLOADS[nm]
        r, tensors = bench_fwd(kata, dev, hip, w, steps, warmup)
        out[nm] = fwd_row(w, r)
        del tensors
        torch.cuda.empty_cache()
    return out


def _cpu_model():
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def _single_thread_rate(workload, seconds):
    """The oracle on one thread (a child process with OMP_NUM_THREADS=1, so the
    OpenMP runtime of this process keeps its setting): evenly spaced rows of
    the workload's heads for about `seconds`, extrapolated like the main
    sample.  Returns (tokens/s, rows, elapsed s)."""
    import subprocess
    code = f"""
import sys, time, json
sys.path.insert(0, {ROOT!r})
import numpy as np, oracle, workloads
w = workloads.WORKLOADS[{workload!r}]
inp = workloads.make_inputs(w, B=1, H=1)  # one head of the same recipe: the rows' cost
orc = oracle.Oracle()
q, k, v = (np.ascontiguousarray(inp[n], dtype=np.float64) for n in ("q", "k", "v"))
BH = w.B * w.H
t0 = time.perf_counter(); orc.fwd_rows(q, k, v, np.zeros(1, np.int64), np.full(1, w.T - 1)); cal = time.perf_counter() - t0
R = max(1, min(int({seconds} / max(cal / w.T * (w.T / 2.0), 1e-12)), w.T))
rows = ((np.arange(R) + 0.5) * w.T / R).astype(np.int64)
bh = np.zeros(R, np.int64)
t0 = time.perf_counter(); orc.fwd_rows(q, k, v, bh, rows); el = time.perf_counter() - t0
units = float(np.sum(rows + 1)); full = BH * w.T * (w.T + 1) / 2.0
print(json.dumps({{"rate": (w.B * w.T) / (el * full / units), "rows": int(R), "elapsed": el,
                  "threads": orc.num_threads()}}))
"""
    env = dict(os.environ, OMP_NUM_THREADS="1")
    r = subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True,
                       timeout=max(120, 8 * seconds))
    if r.returncode != 0:
        return None
    return json.loads(r.stdout.strip().splitlines()[-1])


def cpu_baseline(w, inp, seconds):
    import numpy as np
    import oracle
    orc = oracle.Oracle()
    q = np.ascontiguousarray(inp["q"], dtype=np.float64)
    k = np.ascontiguousarray(inp["k"], dtype=np.float64)
    v = np.ascontiguousarray(inp["v"], dtype=np.float64)
    BH = w.B * w.H
    # calibration: one late row per head
    bh = np.arange(BH)
    tt = np.full(BH, w.T - 1)
    t0 = time.perf_counter()
    orc.fwd_rows(q, k, v, bh, tt)
    cal = time.perf_counter() - t0
    per_unit = cal / float(np.sum(tt + 1))
    # evenly spaced rows per head, sized to about `seconds` of work
    R = int(seconds / max(per_unit * BH * (w.T / 2.0), 1e-12))
    R = max(1, min(R, w.T))
    rows = ((np.arange(R) + 0.5) * w.T / R).astype(np.int64)
    # interleaved batches (each spread over the sequence); a slower host than
    # the calibration suggested stops after about twice `seconds`
    nb = min(R, 8)
    el, sample_units, nrows, rdone = 0.0, 0.0, 0, 0
    for b in range(nb):
        sel = rows[b::nb]
        bh = np.repeat(np.arange(BH), sel.size)
        tt = np.tile(sel, BH)
        t0 = time.perf_counter()
        orc.fwd_rows(q, k, v, bh, tt)
        el += time.perf_counter() - t0
        sample_units += float(np.sum(tt + 1))
        nrows += bh.size
        rdone += sel.size
        if el > 2.0 * seconds:
            break
    full_units = BH * w.T * (w.T + 1) / 2.0
    full_time = el * full_units / sample_units
    single = _single_thread_rate(w.name, max(2.0, seconds / 3.0))
    return {
        "value": (w.B * w.T) / full_time,
        "unit": "tokens/s",
        "cores": orc.num_threads(),
        "kind": "oracle",
        "cpu_model": _cpu_model(),
        "sample": (f"{nrows} rows ({rdone} spread over the sequence per head x {BH} heads) of "
                   f"the fp64 O(T^2) definition on the same inputs, {el:.1f} s on "
                   f"{orc.num_threads()} OpenMP threads; full-workload time extrapolated by the "
                   f"summed row lengths ({full_time:.3g} s)"),
        "single_thread": None if single is None else {
            "value": single["rate"], "unit": "tokens/s", "threads": single["threads"],
            "sample": (f"{single['rows']} evenly spaced rows of head 0 on one thread, "
                       f"{single['elapsed']:.1f} s, extrapolated the same way")},
    }


def bench_decode(kata, dev, hip):
    import numpy as np
    import torch
    import workloads
    w = workloads.WORKLOADS["decode_bf16"]
    inp = workloads.make_inputs(w)
    S, z = kata.prefill_state(upload(inp["k_dev"], "bf16", dev), upload(inp["v_dev"], "bf16", dev))
    sq = upload(inp["steps_q_dev"], "bf16", dev).permute(2, 0, 1, 3).contiguous()
    sk = upload(inp["steps_k_dev"], "bf16", dev).permute(2, 0, 1, 3).contiguous()
    sv = upload(inp["steps_v_dev"], "bf16", dev).permute(2, 0, 1, 3).contiguous()
    out = torch.empty((w.B, w.H, w.dv), dtype=torch.float32, device=dev)
    for s in range(4):  # warm-up on a copy of the state
        kata.decode_step(S.clone(), z.clone(), sq[s], sk[s], sv[s], out=out)
    ev = Events(hip, w.steps + 1)
    stream = torch.cuda.current_stream(dev).cuda_stream
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    hip.hipEventRecord(ev.ev[0], ctypes.c_void_p(stream))
    for s in range(w.steps):
        kata.decode_step(S, z, sq[s], sk[s], sv[s], out=out)
        hip.hipEventRecord(ev.ev[s + 1], ctypes.c_void_p(stream))
    torch.cuda.synchronize()
    el = time.perf_counter() - t0
    per_step = [ev.elapsed(s, s + 1) for s in range(w.steps)]
    ev.close()
    n = w.d * (w.d + 1) // 2
    bytes_step = w.B * w.H * (2 * (n * w.dv + n) * 4 + (2 * w.d + w.dv) * 2 + w.dv * 4)
    avg = sum(per_step) / len(per_step)
    gbs = bytes_step / (avg * 1e-3) / 1e9
    traffic = None
    if os.path.exists(TRAFFIC_FILE):
        with open(TRAFFIC_FILE) as f:
            ent = json.load(f).get("decode_step", {})
        if ent.get("source_sha") == source_sha(("kata_fp32.hip", "kata_common.hpp")):
            traffic = ent.get("hbm_bytes_per_launch")
    return {
        "workload": f"decode_bf16: {w.note}",
        "tokens_per_s": w.B * w.steps / el,
        "ms_per_step": 1e3 * el / w.steps,
        "kernel_ms_per_step": avg,
        "roofline": {"bound": "hbm", "achieved": round(gbs, 1), "peak": PEAK_HBM_GBS,
                     "unit": "GB/s", "frac": round(gbs / PEAK_HBM_GBS, 4),
                     "algorithmic_bytes_per_launch": bytes_step, "traffic": traffic},
    }


def bench_quadratic(kata, dev, Ts=(4096, 16384, 32768), reps=5):
    """Quadratic (flash-style) form against the chunked form at B=1, H=16,
    d=dv=64 (bf16, seeded Gaussian inputs of the long-context recipe), kernel
    time with torch events on the current stream.  MFMA work of the quadratic
    form: the causal half of QK^T and P V, 2*(d+dv) flop per (query, key) pair
    with key <= query."""
    import torch
    import workloads
    rows = []
    for T in Ts:
        inp = workloads.make_inputs("long_bf16", B=1, H=16, T=T)
        q = upload(inp["q_dev"], "bf16", dev)
        k = upload(inp["k_dev"], "bf16", dev)
        v = upload(inp["v_dev"], "bf16", dev)
        out = torch.empty((1, 16, T, 64), dtype=torch.float32, device=dev)
        wq = torch.empty(kata.quadratic_workspace_bytes(1, 16, T, 64, 64, kata.KATA_BF16),
                         dtype=torch.uint8, device=dev)
        # the span given: left to the library, short sequences take the quadratic form too
        span = kata.default_span(1, 16, T, 64, 64, 64, kata.KATA_BF16)
        wc = torch.empty(kata.workspace_bytes(1, 16, T, 64, 64, 64, kata.KATA_BF16, span),
                         dtype=torch.uint8, device=dev)
        ms = {}
        for name, fn in (("quadratic", lambda: kata.fwd_quadratic(q, k, v, out=out, workspace=wq)),
                         ("chunked", lambda: kata.fwd_chunked(q, k, v, 64, span_chunks=span, out=out,
                                                              workspace=wc))):
            for _ in range(2):
                fn()
            torch.cuda.synchronize()
            e0 = torch.cuda.Event(enable_timing=True)
            e1 = torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(reps):
                fn()
            e1.record()
            torch.cuda.synchronize()
            ms[name] = e0.elapsed_time(e1) / reps
        flop = 16 * (T * (T + 1) / 2) * 2 * (64 + 64)
        tf = flop / (ms["quadratic"] * 1e-3) / 1e12
        rows.append({"T": T, "quadratic_ms": round(ms["quadratic"], 4),
                     "chunked_ms": round(ms["chunked"], 4),
                     "quadratic_tokens_per_s": T / (ms["quadratic"] * 1e-3),
                     "chunked_tokens_per_s": T / (ms["chunked"] * 1e-3),
                     "quadratic_mfma": {"achieved": round(tf, 1), "peak": PEAK_BF16_TFLOPS,
                                        "unit": "TFLOP/s", "frac": round(tf / PEAK_BF16_TFLOPS, 4)}})
        del q, k, v, out, wq, wc
    return {"config": "B1 H16 d64 dv64 bf16, C64 for the chunked form", "rows": rows}


def bench_m2(kata, dev, hip, w, q, k, v, steps=10, warmup=3):
    """KATA-M2 (two 32-dim feature blocks) on the same inputs as the headline
    line: stage times from HIP events recorded by the library on the launch
    stream, MFMA rates against the algorithmic work of the M2 feature."""
    import torch
    span = 0
    ws = torch.empty(kata.mg_workspace_bytes(w.B, w.H, w.T, w.d, w.dv, w.C, 2, kata.KATA_BF16,
                                             span), dtype=torch.uint8, device=dev)
    out = torch.empty((w.B, w.H, w.T, w.dv), dtype=torch.float32, device=dev)
    ev = Events(hip, 4 * max(steps, warmup))
    for i in range(warmup):
        kata.mg_fwd_chunked_timed(q, k, v, w.C, 2, ev.block(4 * i), out=out, workspace=ws)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(steps):
        kata.mg_fwd_chunked_timed(q, k, v, w.C, 2, ev.block(4 * i), out=out, workspace=ws)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    names = ("span_state", "scan", "span_output")
    stage = {nm: sum(ev.elapsed(4 * i + j, 4 * i + j + 1) for i in range(steps)) / steps
             for j, nm in enumerate(names)}
    ev.close()
    L = 1024 if w.T >= 1024 else w.T
    alg = algorithmic(w, L, g=2)
    ms = 1e3 * elapsed / steps

    def roof(flop, t_ms):
        tf = flop / (t_ms * 1e-3) / 1e12
        return {"bound": "mfma", "achieved": round(tf, 2), "peak": PEAK_BF16_TFLOPS,
                "unit": "TFLOP/s", "frac": round(tf / PEAK_BF16_TFLOPS, 4)}
    gbs = alg["scan_bytes"] / (stage["scan"] * 1e-3) / 1e9
    return {"feature": "KATA-M2: two blocks of 32 coordinates, n = 2 x 528 packed",
            "tokens_per_s": w.B * w.T / (ms * 1e-3), "ms_per_step": ms,
            "stages_ms": {nm: round(t, 4) for nm, t in stage.items()},
            "stage_roofline": {"span_state": roof(alg["state_flop"], stage["span_state"]),
                               "span_output": roof(alg["output_flop"], stage["span_output"]),
                               "scan": {"bound": "hbm", "achieved": round(gbs, 1),
                                        "peak": PEAK_HBM_GBS, "unit": "GB/s",
                                        "frac": round(gbs / PEAK_HBM_GBS, 4)}},
            "algorithmic_gflop_per_step": round(alg["total_flop"] / 1e9, 2)}


# Paper's tree-scan throughput at B = 1, H = 16, d = 64, C = 128, psi(x) = x on
# an H100 (table of small-batch associative-scan throughput), Mtok/s: context.
PAPER_TREE_SCAN_H100 = {2048: 19.4, 4096: 39.9, 8192: 44.5, 16384: 47.6, 32768: 49.4,
                        65536: 67.5, 131072: 69.4}
LIN_FEATURES = {0: "identity (plain readout)", 1: "relu+eps", 2: "elu+1",
                3: "lorentz lift (n_psi = d + 1)", 4: "lorentz (n_psi = d variant)"}


def lin_bytes(B, H, T, d, dv, L, n=None):
    """Algorithmic HBM bytes of the three linear-feature kernels (bf16 q, k, v;
    fp32 records of S (n x dv) and z (n) per span of L tokens, n = n_psi,
    d by default; fp32 output)."""
    NS = -(-T // L)
    n = d if n is None else n
    rec = B * H * NS * (n * dv + n) * 4
    qk = B * H * T * d * 2
    vv = B * H * T * dv * 2
    return {"span_state": qk + vv + rec, "scan": 2 * rec,
            "span_output": 2 * qk + vv + rec + B * H * T * dv * 4}


def linear_traffic():
    """Calibrated HBM bytes per launch of the psi(x) = x kernels, when the
    counters were taken on the current linear-kernel sources (else {})."""
    if not os.path.exists(TRAFFIC_FILE):
        return {}
    with open(TRAFFIC_FILE) as f:
        lin = json.load(f).get("linear", {})
    if lin.get("source_sha") != source_sha(LIN_SOURCES):
        return {}
    return {k: lin[k]["hbm_bytes_per_launch"] for k in LIN_KERNELS if k in lin}


def bench_linear(kata, dev, hip, steps=10, warmup=3, probe=False):
    """Linear-feature causal linear attention (psi(x) = x and the orthant /
    Lorentz maps) in the state / associative-scan / output pipeline: the
    paper's small-batch associative-scan shape (B1 H16 d64 C128, bf16), per
    feature at T = 131072 with per-stage HBM rooflines, and the T sweep of
    that table for psi(x) = x."""
    import torch
    import workloads
    w = workloads.WORKLOADS["scan_long_bf16"]

    def run(B, H, T, C, feature, q=None, k=None, v=None):
        if q is None:
            inp = workloads.make_inputs(w, B=B, H=H, T=T)
            q, k, v = (upload(inp[n], "bf16", dev) for n in ("q_dev", "k_dev", "v_dev"))
        norm = feature != 0
        span = kata.lin_default_span(B, H, T, w.d, w.dv, C, feature, kata.KATA_BF16)
        ws = torch.empty(max(256, kata.lin_workspace_bytes(B, H, T, w.d, w.dv, C, feature,
                                                           kata.KATA_BF16, span)),
                         dtype=torch.uint8, device=dev)
        out = torch.empty((B, H, T, w.dv), dtype=torch.float32, device=dev)
        ev = Events(hip, 4 * max(steps, warmup))
        for i in range(warmup):
            kata.lin_fwd_chunked(q, k, v, C, feature, 1e-3, norm, span_chunks=span, out=out,
                                 workspace=ws, events=ev.block(4 * i))
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for i in range(steps):
            kata.lin_fwd_chunked(q, k, v, C, feature, 1e-3, norm, span_chunks=span, out=out,
                                 workspace=ws, events=ev.block(4 * i))
        torch.cuda.synchronize()
        ms = 1e3 * (time.perf_counter() - t0) / steps
        names = ("span_state", "scan", "span_output")
        stage = {nm: sum(ev.elapsed(4 * i + j, 4 * i + j + 1) for i in range(steps)) / steps
                 for j, nm in enumerate(names)}
        ev.close()
        return ms, stage, span * C

    inp = workloads.make_inputs(w)
    q, k, v = (upload(inp[n], "bf16", dev) for n in ("q_dev", "k_dev", "v_dev"))
    if probe:  # psi(x) = x only, for the counter runs
        ms, stage, L = run(w.B, w.H, w.T, w.C, 0, q, k, v)
        return {"probe": "linear identity", "ms_per_step": ms, "span_tokens": L}
    traffic = linear_traffic()
    per_feature = {}
    for f, name in LIN_FEATURES.items():
        ms, stage, L = run(w.B, w.H, w.T, w.C, f, q, k, v)
        by = lin_bytes(w.B, w.H, w.T, w.d, w.dv, L, w.d + 1 if f == 3 else w.d)
        roofs = {}
        for nm, t in stage.items():
            gbs = by[nm] / (t * 1e-3) / 1e9
            roofs[nm] = {"bound": "hbm", "achieved": round(gbs, 1), "peak": PEAK_HBM_GBS,
                         "unit": "GB/s", "frac": round(gbs / PEAK_HBM_GBS, 4),
                         "algorithmic_bytes": by[nm],
                         "traffic": traffic.get(nm) if f == 0 else None}
        per_feature[name] = {"tokens_per_s": w.B * w.T / (ms * 1e-3), "ms_per_step": ms,
                             "span_tokens": L,
                             "stages_ms": {nm: round(t, 4) for nm, t in stage.items()},
                             "stage_roofline": roofs}
    del q, k, v
    sweep = []
    for T in sorted(PAPER_TREE_SCAN_H100):
        ms, stage, L = run(1, 16, T, w.C, 0)
        sweep.append({"T": T, "ms": round(ms, 4), "tokens_per_s": T / (ms * 1e-3),
                      "span_tokens": L, "kernel_ms": round(sum(stage.values()), 4),
                      "paper_tree_scan_h100_mtok_s": PAPER_TREE_SCAN_H100[T]})
    return {"workload": f"{w.name}: {w.note}",
            "inputs": "seeded Gaussian q,k (unit rows), v ~ N(0,1), bf16 RNE; eps = 1e-3",
            "kernel_source_sha": source_sha(LIN_SOURCES),
            "features": per_feature, "t_sweep_identity_B1_H16": sweep}


# Paper's linear-state training step (forward + backward) at B = 8, H = 16,
# d = 64, bf16 on an H100 (training-step latency table), ms: context.
PAPER_TRAIN_STEP_H100 = {1024: 10.14, 2048: 20.07, 4096: 39.93, 8192: 79.58}


def bwd_flop(BH, T, d, dv, C):
    """Algorithmic flops of the chunked backward per stage, counted on the
    packed features (n = d(d+1)/2): chunk states 2 C n dv per chunk (forward
    and backward); gradients 4 C n (dv+1) (query- and key-side feature
    cotangents) + 2 C n dv (dv readout) + C^2 (2 dv + 3 d) (in-chunk terms)."""
    n = d * (d + 1) // 2
    NC = -(-T // C)
    chunks = BH * NC
    return {"state": chunks * 2 * C * n * dv,
            "grad": chunks * (4 * C * n * (dv + 1) + 2 * C * n * dv + C * C * (2 * dv + 3 * d))}


def bwd_record_bytes(d, dv):
    """Bytes of one chunk record on the bf16 path (bf16 inputs, d = dv = C =
    64): the state S as bf16 (n dv x 2), then z as fp32 (n x 4)."""
    n = d * (d + 1) // 2
    return n * dv * 2 + n * 4


def bwd_bytes(BH, T, d, dv, C):
    """Algorithmic HBM bytes per launch of the bf16-path backward kernels:
    chunk states write one record per chunk and read the chunk's x (bf16) and
    y rows (v bf16, or a | b fp32) -- also where the launch writes the scanned
    records directly (state and scan in one pass); each scan reads and writes
    every record;
    the gradients read two records, the bf16 q, k, v rows and the fp32 a | b
    rows, and write the fp32 dq, dk, dv rows."""
    NC = -(-T // C)
    R = bwd_record_bytes(d, dv)
    rows_qkv = C * (2 * d + dv) * 2
    rows_ab = C * (dv + 1) * 4
    return {"fwd_states": BH * NC * (R + C * d * 2 + C * dv * 2),
            "bwd_states": BH * NC * (R + C * d * 2 + rows_ab),
            "scan": BH * NC * 2 * R,
            "gradients": BH * NC * (2 * R + rows_qkv + rows_ab + C * (2 * d + dv) * 4)}


def bench_backward(kata, dev, hip, Ts=(1024, 2048, 4096, 8192), steps=5, warmup=2):
    """Training step of KATA-M1 (forward on the bf16 MFMA path saving the row
    denominators D_t, then the O(T) chunked backward taking them) at the
    paper's training-table shape B = 8, H = 16, d = dv = 64, C = 64, bf16
    inputs, fp32 gradients; per-stage HIP-event times of the backward, and the
    HBM rates of its state, scan and gradients kernels against their
    algorithmic bytes (with the bf16 matrix rates of the state and gradients
    kernels beside them)."""
    import torch
    import workloads
    B, H, d, dv, C = 8, 16, 64, 64, 64
    rows = []
    for T in Ts:
        if T == workloads.WORKLOADS["mid_bf16"].T:
            inp = workloads.make_inputs("mid_bf16")
            q, k, v = (upload(inp[nm], "bf16", dev) for nm in ("q_dev", "k_dev", "v_dev"))
            src = "mid_bf16 inputs"
        else:  # same recipe, drawn on the device
            g_ = torch.Generator(device=dev)
            g_.manual_seed(1000 + T)
            q = torch.randn(B, H, T, d, device=dev, generator=g_)
            k = torch.randn(B, H, T, d, device=dev, generator=g_)
            q = (q / q.norm(dim=-1, keepdim=True)).bfloat16().contiguous()
            k = (k / k.norm(dim=-1, keepdim=True)).bfloat16().contiguous()
            v = torch.randn(B, H, T, dv, device=dev, generator=g_).bfloat16().contiguous()
            src = "seeded on device (same recipe)"
        g2 = torch.Generator(device=dev)
        g2.manual_seed(7)
        dout = torch.randn(B, H, T, dv, device=dev, generator=g2)
        fws = torch.empty(kata.workspace_bytes(B, H, T, d, dv, C, kata.KATA_BF16),
                          dtype=torch.uint8, device=dev)
        bws = torch.empty(kata.bwd_workspace_bytes(B, H, T, d, dv, C, 1, kata.KATA_BF16),
                          dtype=torch.uint8, device=dev)
        out = torch.empty((B, H, T, dv), dtype=torch.float32, device=dev)
        den = torch.empty((B, H, T), dtype=torch.float32, device=dev)
        grads = tuple(torch.empty((B, H, T, x), dtype=torch.float32, device=dev)
                      for x in (d, d, dv))
        fev = Events(hip, 2 * max(steps, warmup))
        bev = Events(hip, 7 * max(steps, warmup))
        stream = torch.cuda.current_stream(dev)

        def train_step(i):
            fev.record(2 * i, stream)
            kata.fwd_chunked_train(q, k, v, C, out=out, den=den, workspace=fws)
            fev.record(2 * i + 1, stream)
            kata.bwd_chunked(q, k, v, out, dout, C, 1, workspace=bws, events=bev.block(7 * i),
                             grads=grads, den=den)
        for i in range(warmup):
            train_step(i)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for i in range(steps):
            train_step(i)
        torch.cuda.synchronize()
        ms = 1e3 * (time.perf_counter() - t0) / steps
        names = ("fwd_states", "prefix_scan", "coefficients", "bwd_states", "suffix_scan",
                 "gradients")
        st = {nm: sum(bev.elapsed(7 * i + j, 7 * i + j + 1) for i in range(steps)) / steps
              for j, nm in enumerate(names)}
        # with the state and the scan in one launch per record stream, the scan
        # intervals hold no kernel (their event gaps go to the state stages)
        form = kata.bwd_form(B, H, T, d, dv, C, 1, kata.KATA_BF16)
        quadratic = form == kata.BWD_QUADRATIC  # forms no chunk states: those intervals are empty
        fused = form == kata.BWD_FUSED_STATES
        if quadratic or fused:
            st["fwd_states"] += st.pop("prefix_scan")
            st["bwd_states"] += st.pop("suffix_scan")
        fwd_ms = sum(fev.elapsed(2 * i, 2 * i + 1) for i in range(steps)) / steps
        fev.close()
        bev.close()
        fl = bwd_flop(B * H, T, d, dv, C)

        by = bwd_bytes(B * H, T, d, dv, C)

        def hbm_rate(nbytes, t_ms, flop=None):
            # bf16 inputs at d = dv = C = 64 take the bf16 matrix-core states and
            # gradients; their bound is the records they stream
            gbs = nbytes / (t_ms * 1e-3) / 1e9
            r = {"bound": "hbm", "achieved": round(gbs, 1), "peak": PEAK_HBM_GBS, "unit": "GB/s",
                 "frac": round(gbs / PEAK_HBM_GBS, 4), "algorithmic_bytes": nbytes}
            if flop is not None:
                tf = flop / (t_ms * 1e-3) / 1e12
                r["mfma_bf16"] = {"achieved": round(tf, 1), "peak": PEAK_BF16_TFLOPS,
                                  "unit": "TFLOP/s", "frac": round(tf / PEAK_BF16_TFLOPS, 4)}
            return r
        row = {"T": T, "inputs": src, "train_step_ms": round(ms, 3),
               "forward_ms": round(fwd_ms, 3), "backward_ms": round(sum(st.values()), 3),
               "tokens_per_s": B * T / (ms * 1e-3), "quadratic_backward": quadratic,
               "state_and_scan_fused": fused, "forward_saves_denominators": True,
               "backward_stages_ms": {nm: round(t, 4) for nm, t in st.items()}}
        if quadratic:  # five 64-wide products per causal pair on the matrix cores
            tf = B * H * T * (T + 1) * 5 * d / (st["gradients"] * 1e-3) / 1e12
            row["gradients_roofline"] = {"bound": "mfma_bf16", "achieved": round(tf, 1),
                                         "peak": PEAK_BF16_TFLOPS, "unit": "TFLOP/s",
                                         "frac": round(tf / PEAK_BF16_TFLOPS, 4)}
        else:
            row["gradients_roofline"] = hbm_rate(by["gradients"], st["gradients"], fl["grad"])
            row["bwd_states_roofline"] = hbm_rate(by["bwd_states"], st["bwd_states"], fl["state"])
            row["fwd_states_roofline"] = hbm_rate(by["fwd_states"], st["fwd_states"], fl["state"])
            if not fused:
                row["suffix_scan_roofline"] = hbm_rate(by["scan"], st["suffix_scan"])
        row["paper_linear_state_m1_train_step_h100_ms"] = PAPER_TRAIN_STEP_H100.get(T)
        rows.append(row)
        del fws, bws, out, grads, q, k, v, dout
        torch.cuda.empty_cache()
    return {"config": "KATA-M1 B8 H16 d64 dv64 C64, bf16 inputs, fp32 gradients of "
                      "sum <dout, o> (dout ~ N(0,1))", "rows": rows}


# the KATA-M1 kernels of the d = 64 long-context workload (the M2 and
# quadratic-form instantiations share the names, not the template arguments)
KERNELS = {"span_state": "span_state_kernel<64, 64, 1>",
           "scan": "scan_exclusive_bf16<8, kata::SlotWeight<64, 64, 1> >",
           "span_output": "span_output8_kernel<64, 64, 1>"}
COPY_BYTES = 1 << 30
# the linear-feature kernels of psi(x) = x (plain readout) at d = dv = 64
LIN_KERNELS = {"span_state": "lin_span_state<0>",
               "scan": "scan_exclusive_f32x4<kata::LinUnitWeight",
               "span_output": "lin_span_output<0, false>"}


def copy_probe():
    """A plain device copy of COPY_BYTES, three times: the calibration kernel
    for the FETCH_SIZE / WRITE_SIZE counters."""
    import torch
    src = torch.ones(COPY_BYTES // 2, dtype=torch.bfloat16, device="cuda:0")
    dst = torch.empty_like(src)
    for _ in range(3):
        dst.copy_(src)
    torch.cuda.synchronize()
    print(json.dumps({"copy_probe_bytes": COPY_BYTES, "launches": 3}), flush=True)


def hbm_ceiling(dev, nbytes=COPY_BYTES, reps=10):
    """Practical HBM read+write rate on this GPU: a plain device copy of
    `nbytes` into a second buffer, and an in-place elementwise scale of the same
    buffer (one read and one write per element, the access pattern of the scan
    and of the decode step).  Bytes counted: read + written."""
    import torch
    a = torch.ones(nbytes // 4, dtype=torch.float32, device=dev)
    b = torch.empty_like(a)
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    rates = {}
    for name, op in (("copy", lambda: b.copy_(a)), ("inplace_scale", lambda: a.mul_(1.0))):
        for _ in range(3):
            op()
        torch.cuda.synchronize()
        e0.record()
        for _ in range(reps):
            op()
        e1.record()
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / reps
        rates[name + "_GBps"] = round(2 * nbytes / (ms * 1e-3) / 1e9, 1)
    del a, b
    rates["bytes"] = nbytes
    rates["nominal_GBps"] = PEAK_HBM_GBS
    return rates


def _counter_rows(d):
    import csv
    import glob
    files = glob.glob(os.path.join(d, "**", "*counter_collection.csv"), recursive=True)
    if not files:
        raise SystemExit(f"no counter_collection.csv under {d}")
    rows = []
    for f in files:
        with open(f) as fh:
            rows.extend(csv.DictReader(fh))
    return rows


def _per_dispatch(rows, counter, match):
    """Average over dispatches of the kernels whose name contains `match` of the
    counter (summed over its instances within a dispatch), in KiB."""
    per = {}
    for r in rows:
        if r["Counter_Name"] != counter or match not in r["Kernel_Name"]:
            continue
        per[r["Dispatch_Id"]] = per.get(r["Dispatch_Id"], 0.0) + float(r["Counter_Value"])
    return (sum(per.values()) / len(per), len(per)) if per else (None, 0)


def ingest_traffic(root, workload, span):
    """profiles/traffic_counters.json and its summary from four rocprofv3 --pmc
    runs under `root`: fetch/ and write/ (bench.py) and cfetch/, cwrite/
    (bench.py --copy-probe)."""
    cal = {}
    for cnt, sub in (("FETCH_SIZE", "cfetch"), ("WRITE_SIZE", "cwrite")):
        rows = _counter_rows(os.path.join(root, sub))
        names = {r["Kernel_Name"] for r in rows if r["Counter_Name"] == cnt}
        copies = [n for n in names if "copy" in n.lower()]  # the runtime's copy kernel
        if len(copies) != 1:
            raise SystemExit(f"expected one copy kernel in {sub}, found {sorted(names)}")
        name = copies[0]
        kib, nd = _per_dispatch(rows, cnt, name)
        cal[cnt] = {"copy_kernel": name[:80], "kib_per_dispatch": kib, "dispatches": nd,
                    "factor": COPY_BYTES / (kib * 1024.0)}
    # sections whose counter runs are not under `root` keep their earlier entries
    res = {}
    if os.path.exists(TRAFFIC_FILE):
        with open(TRAFFIC_FILE) as fh:
            res = json.load(fh)
    res["calibration"] = {"copy_bytes": COPY_BYTES, **cal}
    m1 = os.path.isdir(os.path.join(root, "fetch")) and os.path.isdir(os.path.join(root, "write"))
    if m1:
        for key in KERNELS:
            res.pop(key, None)
        res.update({"source_sha": source_sha(), "workload": workload, "span_chunks": span})
    fetch_rows = _counter_rows(os.path.join(root, "fetch")) if m1 else []
    write_rows = _counter_rows(os.path.join(root, "write")) if m1 else []
    for key, match in (KERNELS.items() if m1 else ()):
        fk, nf = _per_dispatch(fetch_rows, "FETCH_SIZE", match)
        wk, nw = _per_dispatch(write_rows, "WRITE_SIZE", match)
        if fk is None or wk is None:
            continue
        fb = fk * 1024.0 * cal["FETCH_SIZE"]["factor"]
        wb = wk * 1024.0 * cal["WRITE_SIZE"]["factor"]
        res[key] = {"fetch_kib_raw": fk, "write_kib_raw": wk, "dispatches": [nf, nw],
                    "fetch_bytes_per_launch": fb, "write_bytes_per_launch": wb,
                    "hbm_bytes_per_launch": fb + wb}
    if os.path.isdir(os.path.join(root, "dfetch")) and os.path.isdir(os.path.join(root, "dwrite")):
        # the decode step (bench.py --decode-probe): 132 launches of decode_step_f32
        fk, nf = _per_dispatch(_counter_rows(os.path.join(root, "dfetch")), "FETCH_SIZE",
                               "decode_step_f32")
        wk, nw = _per_dispatch(_counter_rows(os.path.join(root, "dwrite")), "WRITE_SIZE",
                               "decode_step_f32")
        if fk is not None and wk is not None:
            fb = fk * 1024.0 * cal["FETCH_SIZE"]["factor"]
            wb = wk * 1024.0 * cal["WRITE_SIZE"]["factor"]
            res["decode_step"] = {"fetch_kib_raw": fk, "write_kib_raw": wk, "dispatches": [nf, nw],
                                  "fetch_bytes_per_launch": fb, "write_bytes_per_launch": wb,
                                  "hbm_bytes_per_launch": fb + wb,
                                  "source_sha": source_sha(("kata_fp32.hip", "kata_common.hpp"))}
    if os.path.isdir(os.path.join(root, "lfetch")) and os.path.isdir(os.path.join(root, "lwrite")):
        lres = {"source_sha": source_sha(LIN_SOURCES), "workload": "scan_long_bf16",
                "feature": "identity"}
        fetch_rows = _counter_rows(os.path.join(root, "lfetch"))
        write_rows = _counter_rows(os.path.join(root, "lwrite"))
        for key, match in LIN_KERNELS.items():
            fk, nf = _per_dispatch(fetch_rows, "FETCH_SIZE", match)
            wk, nw = _per_dispatch(write_rows, "WRITE_SIZE", match)
            if fk is None or wk is None:
                continue
            fb = fk * 1024.0 * cal["FETCH_SIZE"]["factor"]
            wb = wk * 1024.0 * cal["WRITE_SIZE"]["factor"]
            lres[key] = {"fetch_kib_raw": fk, "write_kib_raw": wk, "dispatches": [nf, nw],
                         "fetch_bytes_per_launch": fb, "write_bytes_per_launch": wb,
                         "hbm_bytes_per_launch": fb + wb}
        res["linear"] = lres
    with open(TRAFFIC_FILE, "w") as fh:
        json.dump(res, fh, indent=1)
    print(json.dumps(res, indent=1))


def main():
    ap = argparse.ArgumentParser(description=__doc__.splitlines()[0])
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--workload", default="long_bf16")
    ap.add_argument("--span", type=int, default=0, help="span chunks (0 = library default)")
    ap.add_argument("--cpu-seconds", type=float, default=15.0)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-decode", action="store_true")
    ap.add_argument("--no-quadratic", action="store_true")
    ap.add_argument("--no-m2", action="store_true")
    ap.add_argument("--no-linear", action="store_true")
    ap.add_argument("--no-backward", action="store_true")
    ap.add_argument("--linear-probe", action="store_true",
                    help="only run the psi(x) = x linear-feature forward (for rocprofv3 --pmc)")
    ap.add_argument("--copy-probe", action="store_true",
                    help="only run the plain-copy calibration kernel (for rocprofv3 --pmc)")
    ap.add_argument("--decode-probe", action="store_true",
                    help="only run the decode workload (for rocprofv3 --pmc)")
    ap.add_argument("--backward-probe", action="store_true",
                    help="only run the training step at T = 4096 (for rocprofv3 --pmc)")
    ap.add_argument("--no-configs", action="store_true",
                    help="skip the per-workload forward rows (tiny, mid, recall)")
    ap.add_argument("--ingest-traffic", metavar="DIR",
                    help="write profiles/traffic_counters.json from the --pmc runs under DIR")
    args = ap.parse_args()
    if args.ingest_traffic:
        ingest_traffic(args.ingest_traffic, args.workload, args.span or 16)
        return
    world = int(os.environ.get("WORLD_SIZE", "1"))
    if args.gpus != 1 or world != 1:
        print(f"bench.py measures one GPU only (asked for --gpus {args.gpus}, WORLD_SIZE "
              f"{world}); the library has no multi-GPU path (one process drives one GPU).", file=sys.stderr)
        sys.exit(2)

    if args.copy_probe:
        copy_probe()
        return
    if args.linear_probe:
        import paper_2607_17419_amd as kata
        res = bench_linear(kata, "cuda:0", _hip(), steps=3, warmup=1, probe=True)
        print(json.dumps(res), flush=True)
        return
    if args.decode_probe:
        import paper_2607_17419_amd as kata
        res = bench_decode(kata, "cuda:0", _hip())
        print(json.dumps(res), flush=True)
        return
    if args.backward_probe:
        import paper_2607_17419_amd as kata
        res = bench_backward(kata, "cuda:0", _hip(), Ts=(4096,), steps=3, warmup=1)
        print(json.dumps(res), flush=True)
        return

    import numpy as np
    import torch

    import paper_2607_17419_amd as kata
    import workloads

    dev = "cuda:0"
    w = workloads.WORKLOADS[args.workload]
    hip = _hip()
    inp = workloads.make_inputs(w)
    q = upload(inp["q_dev"], w.dtype, dev)
    k = upload(inp["k_dev"], w.dtype, dev)
    v = upload(inp["v_dev"], w.dtype, dev)
    code = kata.KATA_BF16 if w.dtype == "bf16" else kata.KATA_F32
    span = args.span or kata.default_span(w.B, w.H, w.T, w.d, w.dv, w.C, code)
    L = min(span * w.C, -(-w.T // w.C) * w.C)
    out = torch.empty((w.B, w.H, w.T, w.dv), dtype=torch.float32, device=dev)
    ws = torch.empty(kata.workspace_bytes(w.B, w.H, w.T, w.d, w.dv, w.C, code, span),
                     dtype=torch.uint8, device=dev)
    ev = Events(hip, 4 * max(args.steps, args.warmup))
    for i in range(args.warmup):
        kata.fwd_chunked_timed(q, k, v, w.C, ev.block(4 * i), span_chunks=span, out=out,
                               workspace=ws)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(args.steps):
        kata.fwd_chunked_timed(q, k, v, w.C, ev.block(4 * i), span_chunks=span, out=out,
                               workspace=ws)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    stage = {"span_state": 0.0, "scan": 0.0, "span_output": 0.0}
    for i in range(args.steps):
        stage["span_state"] += ev.elapsed(4 * i, 4 * i + 1)
        stage["scan"] += ev.elapsed(4 * i + 1, 4 * i + 2)
        stage["span_output"] += ev.elapsed(4 * i + 2, 4 * i + 3)
    ev.close()
    stage = {kname: t / args.steps for kname, t in stage.items()}
    ms = 1e3 * elapsed / args.steps
    tokens = w.B * w.T
    alg = algorithmic(w, L)

    def mfma_roof(flop, t_ms):
        tf = flop / (t_ms * 1e-3) / 1e12
        return {"bound": "mfma", "achieved": round(tf, 2), "peak": PEAK_BF16_TFLOPS,
                "unit": "TFLOP/s", "frac": round(tf / PEAK_BF16_TFLOPS, 4)}

    roofs = {
        "span_state": mfma_roof(alg["state_flop"], stage["span_state"]),
        "span_output": mfma_roof(alg["output_flop"], stage["span_output"]),
    }
    gbs = alg["scan_bytes"] / (stage["scan"] * 1e-3) / 1e9
    roofs["scan"] = {"bound": "hbm", "achieved": round(gbs, 1), "peak": PEAK_HBM_GBS,
                     "unit": "GB/s", "frac": round(gbs / PEAK_HBM_GBS, 4)}
    dominant = max(stage, key=stage.get)
    roof = dict(roofs[dominant])
    roof["kernel"] = dominant
    roof["traffic"] = None
    sha = source_sha()
    if os.path.exists(TRAFFIC_FILE):
        with open(TRAFFIC_FILE) as f:
            tr = json.load(f)
        ent = tr.get(dominant, {})
        if (tr.get("source_sha") == sha and tr.get("workload") == w.name
                and tr.get("span_chunks") == span and ent):
            roof["traffic"] = ent.get("hbm_bytes_per_launch")

    res = {
        "metric": METRIC,
        "value": tokens / (ms * 1e-3),
        "unit": "tokens/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": w.dtype,
        "data": "synthetic",
        "config": {"workload": f"{w.name}: {w.note}", "B": w.B, "H": w.H, "T": w.T, "d": w.d,
                   "dv": w.dv, "C": w.C, "span_chunks": span, "span_tokens": L,
                   "inputs": "seeded Gaussian q,k (unit rows), v ~ N(0,1), bf16 RNE"},
        "roofline": roof,
        "stages_ms": {kname: round(t, 4) for kname, t in stage.items()},
        "stage_roofline": roofs,
        "mfma_frac_end_to_end": round(alg["total_flop"] / (ms * 1e-3) / 1e12 / PEAK_BF16_TFLOPS, 4),
        "algorithmic_gflop_per_step": round(alg["total_flop"] / 1e9, 2),
        "kernel_source_sha": sha,
    }
    if not args.no_configs:
        res["configs"] = bench_configs(kata, dev, hip)
    if not args.no_decode:
        res["decode"] = bench_decode(kata, dev, hip)
        res["practical_hbm"] = hbm_ceiling(dev)
    if not args.no_m2 and w.d == 64:
        res["m2"] = bench_m2(kata, dev, hip, w, q, k, v)
    if not args.no_quadratic:
        res["quadratic_vs_chunked"] = bench_quadratic(kata, dev)
    if not args.no_linear:
        res["linear_features"] = bench_linear(kata, dev, hip)
    if not args.no_backward:
        res["backward"] = bench_backward(kata, dev, hip)
    if not args.no_cpu_baseline:
        res["cpu_baseline"] = cpu_baseline(w, inp, args.cpu_seconds)
    print(json.dumps(res), flush=True)


def _no_children_left():
    """bench.py starts one child (the single-thread oracle timing, waited for);
    report on stderr and end anything else still attached to this process."""
    try:
        import psutil
    except ImportError:
        return
    kids = psutil.Process().children(recursive=True)
    for p in kids:
        try:
            print(f"bench.py: ending leftover child {p.pid} {p.name()}", file=sys.stderr)
            p.terminate()
        except psutil.Error:
            pass
    psutil.wait_procs(kids, timeout=5)


if __name__ == "__main__":
    try:
        main()
    finally:
        _no_children_left()
