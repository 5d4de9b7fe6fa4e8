#!/usr/bin/env python3
"""Benchmark of the LC-VQ linear layer training step on one MI355X.

A step is one forward (quantise + 2-bit pack, activation transform, matrix-core
product) plus one straight-through backward (dX, dZ, dA, db) of one LC-VQ
weight matrix, through the training pair (the forward saves the backward's
code operand, masks and X', so the backward's prepass handles dY alone), on
seeded synthetic inputs already resident in HBM.  The
reported value is the work of the three products, 6 N m n flop, divided by the
step time.  Prints one JSON line.

  python bench.py [--steps K] [--warmup W] [--workload NAME] [--no-cpu-baseline] [--no-workloads]

By default it also times the larger Llama-shaped workloads (7B MLP, 70B MLP
with the 2-bit pack, a 7B decoder block with AdamW of Z, A and b) for
--workload-steps steps each, the streaming kernels, the packed-codes forward
and the fp64 oracle on the host cores.
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

METRIC = "LC-VQ linear fwd+bwd TFLOP/s (frac of MFMA peak) at 4096x4096; codes bit-exact"
PEAK_MFMA_BF16 = 2500.0      # TFLOP/s, MI355X dense bf16 matrix cores (published)
PEAK_HBM = 8000.0            # GB/s, MI355X HBM3E (published)
DEFAULT_WORKLOAD = "lcvq_4096x4096_n4096_bf16"
MATRIX_KERNELS = ("fwd", "dx", "dw")
OTHER_WORKLOADS = ("lcvq_mlp7b_n8192_bf16", "lcvq_mlp70b_n4096_bf16", "lcvq_block7b_n16384_bf16")


def kernel_source_digest() -> str:
    h = hashlib.sha256()
    for f in sorted(os.listdir(os.path.join(ROOT, "paper_2606_10531_amd", "csrc"))):
        with open(os.path.join(ROOT, "paper_2606_10531_amd", "csrc", f), "rb") as fh:
            h.update(f.encode() + fh.read())
    return h.hexdigest()[:16]


def measured_traffic(kernel: str, workload: str):
    """HBM bytes per launch from the committed rocprofv3 counter summary, if it
    was taken on the current kernel sources; else None."""
    path = os.path.join(ROOT, "profiles", "traffic.json")
    if not os.path.exists(path):
        return None
    try:
        rec = json.load(open(path))
    except ValueError:
        return None
    entry = rec.get(workload, {}).get(kernel)
    if not entry or entry.get("source_digest") != kernel_source_digest():
        return None
    return entry.get("bytes_per_launch")


class Layer:
    """Device buffers and the fwd+bwd step of one LC-VQ weight matrix."""

    def __init__(self, lc, torch, N, m, n, d, k, on_device=False):
        """Inputs from the host generators of the workload recipe, or (on_device)
        drawn on the GPU with the same distributions from a seeded torch
        generator: the larger workloads are only timed here, and drawing
        gigabytes on the host would take longer than timing them."""
        import numpy as np

        import synth
        self.lc, self.N, self.m, self.n, self.d = lc, N, m, n, d
        A, b = synth.draw_map(d, k)
        self.A, self.b = torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda()
        if on_device:
            g = torch.Generator(device="cuda").manual_seed(3000 + k)
            self.inp = None
            self.Z = torch.empty((m, n), device="cuda").uniform_(-0.5, 3.5, generator=g).to(torch.bfloat16)
            self.X = torch.randn((N, n), device="cuda", generator=g).to(torch.bfloat16)
            self.dY = torch.randn((N, m), device="cuda", generator=g).to(torch.bfloat16)
        else:
            inp = synth.layer_inputs(N, m, n, d, "bf16", k=k)
            self.inp = inp

            def dev(bits):
                return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).view(torch.bfloat16).cuda()

            self.Z, self.X, self.dY = dev(inp["Z"]), dev(inp["X"]), dev(inp["dY"])
        bf = torch.bfloat16
        self.Y = torch.empty((N, m), dtype=bf, device="cuda")
        self.packed = torch.empty((m, n // 4), dtype=torch.uint8, device="cuda")
        self.dX = torch.empty((N, n), dtype=bf, device="cuda")
        self.dZ = torch.empty((m, n), dtype=bf, device="cuda")
        self.dA = torch.empty((d, d), dtype=torch.float32, device="cuda")
        self.db = torch.empty((d,), dtype=torch.float32, device="cuda")
        self.wsf = torch.empty(lc.workspace_bytes(lc.OP_FWD, N, m, n, d, bf), dtype=torch.uint8, device="cuda")
        self.wsb = torch.empty(lc.workspace_bytes(lc.OP_BWD, N, m, n, d, bf), dtype=torch.uint8, device="cuda")
        # the training pair's saved state: the forward writes the backward's code
        # operand, masks and X' once, and the backward's prepass handles dY alone
        self.saved = lc.new_saved(N, m, n, d, bf, "cuda")

    def step(self):
        """The training pair: lcvq_linear_fwd_train (with the 2-bit pack) + lcvq_linear_bwd_train."""
        lc = self.lc
        lc.linear_fwd(self.Z, self.A, self.b, self.X, self.d, packed_out=self.packed, workspace=self.wsf,
                      out=self.Y, saved=self.saved)
        lc.linear_bwd(self.Z, self.A, self.b, self.X, self.dY, self.d, dX=self.dX, dZ=self.dZ, dA=self.dA,
                      db=self.db, workspace=self.wsb, saved=self.saved)

    def step_plain(self):
        """The same step through the plain calls (the backward rebuilds codes, mask and X')."""
        lc = self.lc
        lc.linear_fwd(self.Z, self.A, self.b, self.X, self.d, packed_out=self.packed, workspace=self.wsf,
                      out=self.Y)
        lc.linear_bwd(self.Z, self.A, self.b, self.X, self.dY, self.d, dX=self.dX, dZ=self.dZ, dA=self.dA,
                      db=self.db, workspace=self.wsb)

    def step_dge(self, k=5.0, cap=3.0):
        """The same step with the differentiable gradient estimator in the backward."""
        lc = self.lc
        lc.linear_fwd(self.Z, self.A, self.b, self.X, self.d, packed_out=self.packed, workspace=self.wsf,
                      out=self.Y, saved=self.saved)
        lc.linear_bwd_dge(self.Z, self.A, self.b, self.X, self.dY, self.d, k=k, cap=cap, dX=self.dX, dZ=self.dZ,
                          dA=self.dA, db=self.db, workspace=self.wsb, saved=self.saved)

    def step_xavier(self):
        """The same step with the latent in the Xavier domain (Sec. 3.4): the same
        latents read as W_p, quantised through W_p / s' + t."""
        lc = self.lc
        qs, qb = lc.xavier_quantizer(self.m, self.n)
        lc.linear_fwd(self.Z, self.A, self.b, self.X, self.d, packed_out=self.packed, workspace=self.wsf,
                      out=self.Y, q_scale=qs, q_shift=qb, saved=self.saved)
        lc.linear_bwd(self.Z, self.A, self.b, self.X, self.dY, self.d, dX=self.dX, dZ=self.dZ, dA=self.dA,
                      db=self.db, workspace=self.wsb, q_scale=qs, q_shift=qb, saved=self.saved)

    def flops(self):
        return 6.0 * self.N * self.m * self.n


def timer_read(lib, kernel_id):
    ms, cnt = ctypes.c_double(), ctypes.c_int64()
    lib.lcvq_timer_read(kernel_id, ctypes.byref(ms), ctypes.byref(cnt))
    return ms.value, cnt.value


def hbm_kernels(lc, torch):
    """Achieved bandwidth of the streaming kernels on a 28672 x 8192 matrix
    (470 MB of bf16 latents, larger than the 256 MB last-level cache)."""
    import numpy as np

    import synth
    m, n, d = 28672, 8192, 8
    lib = lc._lib.load()
    Z = torch.from_numpy(synth.draw_latent(m, n, 0, "bf16").view(np.int16)).view(torch.bfloat16).cuda()
    A, b = torch.eye(d, device="cuda"), torch.zeros(d, device="cuda")
    packed = torch.empty((m, n // 4), dtype=torch.uint8, device="cuda")
    W = torch.empty((m, n), dtype=torch.bfloat16, device="cuda")
    # AdamW on the same matrix: fp32 master, moments; bf16 gradient and bf16 latent copy
    theta = Z.float().reshape(-1)
    m1, m2 = torch.zeros_like(theta), torch.zeros_like(theta)
    gZ = W.reshape(-1)
    shadow = torch.empty_like(gZ)
    out = {}
    cases = [("pack2bit_from_bf16", lambda: lc.pack2bit(Z, out=packed), 2.25, "pack"),
             ("dequant_packed_to_bf16", lambda: lc.dequant(packed, A, b, d, n=n, src_kind=lc.SRC_PACKED2,
                                                           out=W), 2.25, "dequant"),
             ("dequant_bf16_latent_to_bf16", lambda: lc.dequant(Z, A, b, d, out=W), 4.0, "dequant"),
             # LC encode of a dense bf16 weight into packed codes (reads W, writes 2 bits per element)
             ("encode_bf16_to_packed", lambda: lc._lib.check(lib.lcvq_encode(
                 m, n, d, W.data_ptr(), lc._lib.BF16, A.data_ptr(), b.data_ptr(), None, packed.data_ptr(),
                 lc._stream(W.device)), "lcvq_encode"), 2.25, "encode"),
             # per parameter: theta, m1, m2 read + written (24 B), bf16 gradient read, bf16 copy written
             ("adamw_step_fp32_master_bf16_grad",
              lambda: lc.adamw_step(theta, gZ, m1, m2, 1, 1e-4, shadow=shadow), 28.0, "adam")]
    for name, fn, bpe, kname in cases:
        for _ in range(3):
            fn()
        torch.cuda.synchronize()
        kid = lc._lib.KERNELS.index(kname)
        lib.lcvq_timer_enable(1 << kid)
        for _ in range(20):
            fn()
        torch.cuda.synchronize()
        ms, cnt = timer_read(lib, kid)
        lib.lcvq_timer_enable(0)
        us = 1e3 * ms / max(cnt, 1)
        gbps = bpe * m * n / (us * 1e-6) / 1e9
        out[name] = {"us": round(us, 2), "GB/s": round(gbps, 1), "frac_hbm": round(gbps / PEAK_HBM, 3),
                     "bytes_per_elem": bpe, "shape": [m, n]}
    del Z, packed, W, theta, m1, m2, shadow
    return out


def variant_step(lc, torch, layers, steps, which, label):
    """fwd + bwd with a variant of the method (`which`: a Layer method), timed like
    the main step, with its weight-gradient kernel."""
    lib = lc._lib.load()

    def step():
        for L in layers:
            getattr(L, which)()

    for _ in range(3):
        step()
    start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    start.record()
    for _ in range(steps):
        step()
    stop.record()
    torch.cuda.synchronize()
    ms = start.elapsed_time(stop) / steps
    lib.lcvq_timer_enable((1 << len(lc._lib.KERNELS)) - 1)
    for _ in range(20):
        step()
    torch.cuda.synchronize()
    kernels = {}
    for kid, name in enumerate(lc._lib.KERNELS):
        k_ms, cnt = timer_read(lib, kid)
        if cnt:
            kernels[name] = round(1e3 * k_ms / 20, 2)
    lib.lcvq_timer_enable(0)
    flops = sum(L.flops() for L in layers)
    return {"variant": label, "ms_per_step": round(ms, 4), "TFLOP/s": round(flops / (ms * 1e-3) / 1e12, 2),
            "kernels_us_per_step": kernels}


def workload_steps(lc, torch, names, steps):
    """The fwd + bwd step on the other Llama-shaped workloads (every matrix of
    the workload in turn on one stream), timed like the main step.  The 7B
    decoder block also runs the AdamW update of each matrix's latent (fp32
    master, bf16 copy used by the next forward) and of its map A and offset b,
    inside the timed step, as one training step would."""
    import synth
    out = {}
    for name in names:
        wl = synth.WORKLOADS[name]
        layers = [Layer(lc, torch, wl["N"], m, n, wl["d"], k, on_device=True) for k, (m, n) in enumerate(wl["mats"])]
        adam = name.startswith("lcvq_block7b")
        states = []
        if adam:
            for L in layers:
                th = {"Z": L.Z.float(), "A": L.A, "b": L.b}   # A and b are updated in place
                states.append({key: (t, torch.zeros_like(t), torch.zeros_like(t)) for key, t in th.items()})
        count = [0]

        def step():
            for L in layers:
                L.step()
            if adam:
                count[0] += 1
                for L, st in zip(layers, states):
                    for key, grad, shadow in (("Z", L.dZ, L.Z), ("A", L.dA, None), ("b", L.db, None)):
                        th, m1, m2 = st[key]
                        lc.adamw_step(th, grad.reshape(-1), m1.reshape(-1), m2.reshape(-1), count[0], 1e-4,
                                      shadow=None if shadow is None else shadow.reshape(-1))

        for _ in range(3):
            step()
        start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        start.record()
        for _ in range(steps):
            step()
        stop.record()
        torch.cuda.synchronize()
        ms = start.elapsed_time(stop) / steps
        flops = sum(L.flops() for L in layers)
        out[name] = {"N": wl["N"], "matrices": [list(x) for x in wl["mats"]], "ms_per_step": round(ms, 3),
                     "TFLOP/s": round(flops / (ms * 1e-3) / 1e12, 2),
                     "frac_of_peak": round(flops / (ms * 1e-3) / 1e12 / PEAK_MFMA_BF16, 4),
                     "step": "training pair: fwd (+2-bit pack) + straight-through bwd" + (" + AdamW of Z, A, b" if adam else "")}
        del layers, states
        torch.cuda.empty_cache()
    return out


def packed_decode(lc, torch, token_counts=(1, 4, 16)):
    """Layer output from packed 2-bit codes (inference) for decode-sized batches,
    on 28672 x 8192 and 8192 x 28672 matrices, four of each (470 MB of codes,
    more than the 256 MB last-level cache), called in turn.  Algorithmic bytes
    per call: the codes (m n / 4), X (N n bf16) and Y (N m bf16)."""
    import synth
    d = 8
    lib = lc._lib.load()
    mats = [(28672, 8192), (8192, 28672)] * 4
    g = torch.Generator(device="cuda").manual_seed(0)
    P = [torch.randint(0, 256, (m, n // 4), dtype=torch.uint8, device="cuda", generator=g) for m, n in mats]
    A, b = [torch.from_numpy(x).cuda() for x in synth.draw_map(d, 0)]
    kp, kq = lc._lib.KERNELS.index("packed"), lc._lib.KERNELS.index("packed_prep")
    out = {}
    for N in token_counts:
        X = {n: torch.randn(N, n, device="cuda", generator=g).to(torch.bfloat16) for n in (8192, 28672)}
        Y = [torch.empty((N, m), dtype=torch.bfloat16, device="cuda") for m, _ in mats]
        ws = [torch.empty(lc.workspace_bytes(lc.OP_FWD_PACKED, N, m, n, d, torch.bfloat16), dtype=torch.uint8,
                          device="cuda") for m, n in mats]

        def run():
            for i, (m, n) in enumerate(mats):
                lc.linear_fwd_packed(P[i], A, b, X[n], d, out=Y[i], workspace=ws[i])

        for _ in range(3):
            run()
        start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        start.record()
        for _ in range(20):
            run()
        stop.record()
        torch.cuda.synchronize()
        call_us = 1e3 * start.elapsed_time(stop) / (20 * len(mats))
        lib.lcvq_timer_enable((1 << kp) | (1 << kq))
        for _ in range(10):
            run()
        torch.cuda.synchronize()
        pm, pc = timer_read(lib, kp)
        qm, qc = timer_read(lib, kq)
        lib.lcvq_timer_enable(0)
        pus, qus = 1e3 * pm / max(pc, 1), 1e3 * qm / max(qc, 1)
        nbytes = sum(m * n / 4 + 2 * N * (n + m) for m, n in mats) / len(mats)
        gbps = nbytes / (pus * 1e-6) / 1e9
        out[f"N{N}"] = {"product_us": round(pus, 2), "prepass_us": round(qus, 2),
                        "prepass_launches_per_call": round(qc / max(pc, 1), 2), "call_us": round(call_us, 2),
                        "GB/s": round(gbps, 1), "frac_hbm": round(gbps / PEAK_HBM, 3),
                        "bytes_per_call": int(nbytes)}
    out["shapes"] = [[28672, 8192], [8192, 28672]]
    out["note"] = ("GB/s and frac_hbm over the product kernel's average duration; call_us includes the prepass, "
                   "which is launched only where the product blocks do not compute X'' themselves")
    del P
    return out


def step_distribution(torch, step, K):
    """Per-step times of K more steps, each between its own pair of events
    (reported beside the K-step mean, which comes from a run without them)."""
    evs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(K)]
    torch.cuda.synchronize()
    for s, e in evs:
        s.record()
        step()
        e.record()
    torch.cuda.synchronize()
    t = sorted(s.elapsed_time(e) for s, e in evs)
    return {"median_ms": round(t[len(t) // 2], 4), "min_ms": round(t[0], 4), "max_ms": round(t[-1], 4), "steps": K}


def sample_sclk(torch, step, seconds=2.5):
    """Shader clock while steps keep the GPU busy, from a helper thread: the
    level the driver marks as current in sysfs (pp_dpm_sclk), and, where the
    amdsmi module is importable, the power-management firmware's current
    graphics clock of each XCD and the socket power (readings from the first
    second are dropped: the firmware's figures lag the load).  Plain reads: no
    helper program is started; None where nothing is readable."""
    import glob
    import re
    import threading
    import time
    files = sorted(glob.glob("/sys/class/drm/card*/device/pp_dpm_sclk"))
    smi = None
    try:
        import amdsmi
        amdsmi.amdsmi_init()
        handles = amdsmi.amdsmi_get_processor_handles()
        smi = (amdsmi, handles[0]) if handles else None
    except Exception:
        smi = None
    levels, xcd_clocks, power = [], [], []

    def probe():
        t_start = time.time()
        while time.time() - t_start < seconds - 0.1:
            time.sleep(0.25)
            for f in files:
                try:
                    m = re.search(r"(\d+)\s*mhz\s*\*", open(f).read(), re.IGNORECASE)
                except OSError:
                    continue
                if m:
                    levels.append(int(m.group(1)))
            if smi is not None and time.time() - t_start > 1.0:
                try:
                    met = smi[0].amdsmi_get_gpu_metrics_info(smi[1])
                    clk = [int(c) for c in met.get("current_gfxclks", []) if isinstance(c, int) and 0 < c < 10000]
                    if clk:
                        xcd_clocks.append(clk)
                    pw = met.get("current_socket_power")
                    if isinstance(pw, int) and pw > 0:
                        power.append(pw)
                except Exception:
                    pass

    th = threading.Thread(target=probe)
    th.start()
    t0 = time.time()
    while th.is_alive() and time.time() - t0 < seconds + 1.0:
        for _ in range(20):
            step()
        torch.cuda.synchronize()
    th.join()
    if smi is not None:
        try:
            smi[0].amdsmi_shut_down()
        except Exception:
            pass
    out = {"sclk_mhz": max(levels) if levels else None, "source": "sysfs pp_dpm_sclk (current level) during steps"}
    if xcd_clocks:
        mean = sum(sum(c) / len(c) for c in xcd_clocks) / len(xcd_clocks)
        out["gfxclk_mhz"] = round(mean, 1)
        out["gfxclk_mhz_per_xcd_last"] = xcd_clocks[-1]
        out["socket_power_w"] = round(sum(power) / len(power), 1) if power else None
        out["gfxclk_source"] = ("amdsmi gpu metrics current_gfxclks (mean over XCDs and over the readings "
                                "after the first second of steps)")
    return out


def library_gemm(torch, N, m, n):
    """Context: one plain bf16 product of the same shape (Y = X W^T, N(0,1) data)
    through torch.matmul, i.e. the vendor GEMM library, with no quantisation."""
    g = torch.Generator(device="cuda").manual_seed(0)
    X = torch.randn(N, n, device="cuda", generator=g).to(torch.bfloat16)
    W = torch.randn(m, n, device="cuda", generator=g).to(torch.bfloat16)
    for _ in range(5):
        torch.matmul(X, W.t())
    start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    start.record()
    for _ in range(20):
        torch.matmul(X, W.t())
    stop.record()
    torch.cuda.synchronize()
    us = 1e3 * start.elapsed_time(stop) / 20
    return {"op": "torch.matmul bf16 X[N,n] @ W[m,n]^T", "shape": [N, m, n], "us": round(us, 2),
            "TFLOP/s": round(2.0 * N * m * n / (us * 1e-6) / 1e12, 1)}


def cpu_baseline(layer, max_seconds: float):
    """The fp64 oracle on the host, on the same inputs (a bounded number of full
    fwd+bwd repetitions), with its parity check of the GPU results."""
    import numpy as np
    import torch

    import oracle as orc
    try:
        from threadpoolctl import threadpool_info
        cores = max([p.get("num_threads", 1) for p in threadpool_info() if p.get("user_api") == "blas"] or [1])
    except Exception:  # pragma: no cover
        cores = os.cpu_count()
    inp, d = layer.inp, layer.d
    v = {k: orc.widen(inp[k], "bf16") for k in ("Z", "X", "dY")}
    A64, b64 = inp["A"].astype(np.float64), inp["b"].astype(np.float64)
    reps, t0 = 0, time.perf_counter()
    while True:
        Yref, codes = orc.linear_forward(v["Z"], A64, b64, v["X"], d)
        ref = orc.linear_backward(v["Z"], A64, b64, v["X"], v["dY"], d)
        reps += 1
        el = time.perf_counter() - t0
        if el >= max_seconds or reps >= 200:
            break
    per = el / reps

    def host(t):
        t = t.detach().cpu()
        if t.dtype == torch.bfloat16:
            return orc.widen(t.view(torch.int16).numpy().view(np.uint16), "bf16")
        return t.numpy().astype(np.float64)

    def rel(a, r):
        return float(np.linalg.norm(a - r) / np.linalg.norm(r))

    layer.step()
    torch.cuda.synchronize()
    parity = {"codes_bit_exact": bool(np.array_equal(layer.packed.cpu().numpy(), orc.pack2bit(codes))),
              "rel_fro": {"Y": rel(host(layer.Y), Yref), "dX": rel(host(layer.dX), ref["dX"]),
                          "dZ": rel(host(layer.dZ), ref["dZ"]), "dA": rel(host(layer.dA), ref["dA"]),
                          "db": rel(host(layer.db), ref["db"])},
              "tolerance": 2e-2}
    model = None
    try:
        for line in open("/proc/cpuinfo"):
            if line.lower().startswith("model name"):
                model = line.split(":", 1)[1].strip()
                break
    except OSError:
        pass
    return {"value": round(layer.flops() / per / 1e12, 5), "unit": "TFLOP/s", "cores": cores,
            "nproc": len(os.sched_getaffinity(0)), "cpu_model": model, "kind": "oracle",
            "sample": f"full {layer.m}x{layer.n} layer, {layer.N} tokens, fwd+bwd in fp64 (numpy/OpenBLAS), "
                      f"{reps} repetition(s), {per:.2f} s each",
            "parity": parity}


def main():
    ap = argparse.ArgumentParser(description=__doc__, formatter_class=argparse.RawDescriptionHelpFormatter)
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--workload", default=DEFAULT_WORKLOAD)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-hbm", action="store_true")
    ap.add_argument("--no-workloads", action="store_true",
                    help="skip the larger Llama-shaped workloads (7B MLP, 70B MLP + pack, 7B block with AdamW)")
    ap.add_argument("--workload-steps", type=int, default=10)
    ap.add_argument("--cpu-seconds", type=float, default=10.0)
    ap.add_argument("--copy-probe", type=int, default=0, metavar="BYTES",
                    help="only run a plain device-to-device copy of BYTES (counter calibration) and exit")
    args = ap.parse_args()
    if args.copy_probe:
        import torch
        src = torch.ones(args.copy_probe // 4, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"copy_probe_bytes": args.copy_probe, "launches": 3}))
        return
    if args.gpus != 1:
        print(f"bench.py: this build runs on one GPU only (asked for --gpus {args.gpus}); the multi-GPU "
              "sharding of the layer is not built.", file=sys.stderr)
        sys.exit(2)

    import torch

    import paper_2606_10531_amd as lc
    import synth
    assert torch.cuda.is_available(), "bench.py needs a GPU"
    lib = lc._lib.load()
    wl = synth.WORKLOADS[args.workload]
    if wl["dtype"] != "bf16":
        sys.exit("bench.py times the bf16 matrix-core path; pick a bf16 workload")
    layers = [Layer(lc, torch, wl["N"], m, n, wl["d"], k) for k, (m, n) in enumerate(wl["mats"])]

    def step():
        for L in layers:
            L.step()

    # per-kernel breakdown first (untimed): at least 250 steps with every kernel
    # launch bracketed by HIP events on its stream (the library's timer).  The
    # breakdown and the dominant kernel's average launch time come from this one
    # run, so the breakdown sums to no more than this run's step time; the run
    # also brings the chip to its loaded clocks before the timed region (the
    # extra event records lengthen the step a little, which is why `value` comes
    # from the run below)
    k_ev = max(args.steps, 250)
    lib.lcvq_timer_enable((1 << len(lc._lib.KERNELS)) - 1)
    start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    start.record()
    for _ in range(k_ev):
        step()
    stop.record()
    torch.cuda.synchronize()
    ms_step_ev = start.elapsed_time(stop) / k_ev
    breakdown, launch_us, launches = {}, {}, {}
    for kid, name in enumerate(lc._lib.KERNELS):
        ms, cnt = timer_read(lib, kid)
        if cnt:
            breakdown[name] = round(1e3 * ms / k_ev, 2)       # us per step
            launch_us[name] = 1e3 * ms / cnt
            launches[name] = cnt
    lib.lcvq_timer_enable(0)
    dominant = max(MATRIX_KERNELS, key=lambda k: breakdown.get(k, 0.0))
    # the dominant kernel's average launch time from a second run in which only
    # its launches are bracketed by events (one pair per step: the least
    # perturbation of the kernels around it)
    k_dom = max(args.steps, 100)
    dom_kid = list(lc._lib.KERNELS).index(dominant)
    timer_read(lib, dom_kid)  # clear
    lib.lcvq_timer_enable(1 << dom_kid)
    for _ in range(k_dom):
        step()
    torch.cuda.synchronize()
    ms_dom, dom_cnt = timer_read(lib, dom_kid)
    lib.lcvq_timer_enable(0)
    dom_us = 1e3 * ms_dom / dom_cnt

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()

    # timed region: K steps between two events, nothing else recorded
    torch.cuda.synchronize()
    start.record()
    for _ in range(args.steps):
        step()
    stop.record()
    torch.cuda.synchronize()
    ms_step = start.elapsed_time(stop) / args.steps

    dist = step_distribution(torch, step, args.steps)
    sclk = sample_sclk(torch, step)

    flops = sum(L.flops() for L in layers)
    value = flops / (ms_step * 1e-3) / 1e12
    per_launch_flop = 2.0 * sum(L.N * L.m * L.n for L in layers) / len(layers)
    achieved = per_launch_flop / (dom_us * 1e-6) / 1e12
    traffic = measured_traffic(dominant, args.workload)

    res = {
        "metric": METRIC, "value": round(value, 2), "unit": "TFLOP/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": round(ms_step, 4), "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "bf16", "data": "synthetic",
        "config": {"workload": args.workload, "N": wl["N"], "matrices": [list(x) for x in wl["mats"]],
                   "d": wl["d"], "step": "training pair: fwd (+2-bit pack, saving codes, masks and X' for "
                                         "the backward) + straight-through bwd (dX, dZ, dA, db)",
                   "saved_state_bytes": int(layers[0].saved.numel())},
        "frac_of_peak": round(value / PEAK_MFMA_BF16, 4),
        "roofline": {"kernel": dominant, "bound": "mfma", "achieved": round(achieved, 2),
                     "peak": PEAK_MFMA_BF16, "unit": "TFLOP/s", "frac": round(achieved / PEAK_MFMA_BF16, 4),
                     "traffic": traffic, "avg_launch_us": round(dom_us, 2), "launches": dom_cnt,
                     "flop_per_launch": per_launch_flop, "ms_per_step_with_kernel_events": round(ms_step_ev, 4),
                     "avg_launch_note": (f"{k_dom} untimed steps with only this kernel's launches bracketed by HIP "
                                         "events on its stream; the interval includes its dispatch and the "
                                         "end-of-kernel write-back that a profiler's kernel record leaves out")},
        "kernels_us_per_step": breakdown,
        "kernels_us_per_step_note": (f"every launch bracketed by HIP events over {k_ev} untimed steps run just "
                                     "before the warm-up and the timed region; sums to at most "
                                     "ms_per_step_with_kernel_events"),
        "step_distribution": dist,
        "gpu_clock": sclk,
        "frac_of_peak_at_measured_clock": (round(value / (PEAK_MFMA_BF16 * sclk["gfxclk_mhz"] / 2400.0), 4)
                                           if sclk and sclk.get("gfxclk_mhz") else None),
    }
    res["plain_step"] = variant_step(lc, torch, layers, args.steps, "step_plain",
                                     "the plain calls: the backward rebuilds codes, mask and X' from Z and X")
    res["dge_step"] = variant_step(lc, torch, layers, args.steps, "step_dge",
                                   "differentiable gradient estimator, k=5, slope cap 3, latent mask")
    res["xavier_step"] = variant_step(lc, torch, layers, args.steps, "step_xavier",
                                      "latent in the Xavier domain: codes of W_p / s' + t, gradient / s'")
    if not args.no_workloads:
        res["workloads"] = workload_steps(lc, torch, [w for w in OTHER_WORKLOADS if w != args.workload],
                                          args.workload_steps)
    L0 = layers[0]
    res["library_gemm_same_shape"] = library_gemm(torch, L0.N, L0.m, L0.n)
    if not args.no_hbm:
        res["hbm_kernels"] = hbm_kernels(lc, torch)
        res["packed_decode"] = packed_decode(lc, torch)
    if not args.no_cpu_baseline:
        res["cpu_baseline"] = cpu_baseline(layers[0], args.cpu_seconds)
        res["cpu_baseline"]["note"] = "first matrix of the workload" if len(layers) > 1 else "whole workload"
    print(json.dumps(res), flush=True)


if __name__ == "__main__":
    main()
