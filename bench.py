#!/usr/bin/env python3
"""Throughput of the beyond-Limber C_l hot path on one MI355X.

Workload: a batch of parameter points, each a full set of 15 tracers (10 clustering + 5
lensing bins, 120 spectra) x 103 multipoles in [2, 2000], N_k = N_chi = 1024, FP32, every
point with its own cosmology (chi(z), D(z), P(k)) and biases.  Inputs are seeded synthetic
and resident in HBM before timing.  A step is one call of the whole hot path over the batch:
kernel assembly, FFTLog coefficients, windows and projection (forward), then the adjoint
to dP, db, dn(z) and dD(z) with the windows recomputed (backward).

Prints one JSON line.  `value` is C_l sets per second for forward + backward (a set = 120
spectra x 103 l); the forward-only rate is reported beside it.
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_FP32_VECTOR_TFLOPS = 157.3  # MI355X, 256 CUs at 2.4 GHz
PEAK_HBM_GBS = 8000.0


def fused_kernel_flops(T, L, B, N, n_k):
    """Algorithmic flops of one launch of the windows + projection kernel.

    Per (point, multipole): T inverse real FFTs of length N (2.5 N log2 N each), the complex
    product c_n U_l(n) over N/2 coefficients (6 flops each), the k scaling (2 per node) and
    the symmetric projection sum_j s_j W_i W_j over T(T+1)/2 pairs (2 flops per node).
    """
    import math
    per = T * (2.5 * N * math.log2(N) + 6 * (N // 2) + 2 * n_k) + T * (T + 1) // 2 * 2 * n_k
    return per * L * B


def bwd_kernel_flops(T, L, B, N, n_k):
    """Algorithmic flops of one launch of the backward windows kernel.

    Per (point, multipole): the forward windows again (T inverse FFTs and the U product),
    Y = G W (2 T^2 per node), sum_t W Y (2 T per node), the scaled cotangent (4 T per node),
    T forward real FFTs of the cotangent and the product with conj(U) accumulated (8 per
    coefficient).
    """
    import math
    fft = 2.5 * N * math.log2(N)
    per = T * (2 * fft + 6 * (N // 2) + 8 * (N // 2) + 6 * n_k) + 2 * T * T * n_k
    return per * L * B


KERNEL_SOURCES = ["paper_2505_22718_amd/csrc/backward.hip", "paper_2505_22718_amd/csrc/common.h",
                  "paper_2505_22718_amd/csrc/internal.h", "paper_2505_22718_amd/csrc/xcd_map.h"]
TRAFFIC_RECORD = os.path.join(ROOT, "profiles", "pmc_k_bwd_windows_cfg1_batch256.md")
# the same for the forward windows + projection kernel
FWD_KERNEL_SOURCES = ["paper_2505_22718_amd/csrc/forward.hip", "paper_2505_22718_amd/csrc/common.h",
                      "paper_2505_22718_amd/csrc/internal.h", "paper_2505_22718_amd/csrc/sched_layout.h",
                      "paper_2505_22718_amd/csrc/xcd_map.h"]
FWD_TRAFFIC_RECORD = os.path.join(ROOT, "profiles", "pmc_k_windows_cl_cfg1_batch256.md")
PEAK_HBM_GBPS = 8000.0
PEAK_FP32_MFMA_TFLOPS = 157.3


def sources_digest():
    """SHA-256 over the sources of the dominant kernel (a counter record is valid for one digest)."""
    import hashlib
    h = hashlib.sha256()
    for rel in KERNEL_SOURCES:
        with open(os.path.join(ROOT, rel), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def fwd_sources_digest():
    """SHA-256 over the forward windows kernel's sources."""
    import hashlib
    h = hashlib.sha256()
    for rel in FWD_KERNEL_SOURCES:
        with open(os.path.join(ROOT, rel), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def _read_record(path):
    rec = None
    if os.path.exists(path):
        with open(path) as fh:
            for line in fh:
                if line.startswith("traffic-record: "):
                    rec = json.loads(line[len("traffic-record: "):])
    return rec


def fwd_traffic_bytes(batch, launch):
    """HBM bytes per launch of k_windows_cl from its committed counter record, under the same
    rules as traffic_bytes (its sources, the batch, and the forward launch mode)."""
    rec = _read_record(FWD_TRAFFIC_RECORD)
    if not rec or rec.get("sources_sha256") != fwd_sources_digest():
        return None
    if rec.get("batch") != batch or rec.get("launch", {}).get("fwd_mode") != launch["fwd_mode"]:
        return None
    return rec["hbm_bytes_per_launch"]


def contraction_flops(T, L, B, n_k):
    """Flops of the projection C = W diag(s) W^T in one windows launch: algorithmic (the T(T+1)/2
    pairs, 2 per node) and as issued on MFMA (the full 16 x 16 Gram tile per (point, multipole))."""
    return T * (T + 1) * n_k * L * B, 2 * 16 * 16 * n_k * L * B


def traffic_bytes(batch, launch):
    """HBM bytes per launch of k_bwd_windows from the committed rocprofv3 counter record
    (FETCH_SIZE and WRITE_SIZE, each scaled by what the counter reads for a plain copy of known
    size), or None if there is none, if the kernel's sources changed since it was taken, or if the
    launch being timed is not the one it was taken on: the batch and the launch shape (the number
    of multipole chunks per point, set by bwd_chunk_mul, and the packed adjoint's two halves per
    chunk, bwd_pack, set how many partial rows are written)."""
    if not os.path.exists(TRAFFIC_RECORD):
        return None
    rec = None
    with open(TRAFFIC_RECORD) as fh:
        for line in fh:
            if line.startswith("traffic-record: "):
                rec = json.loads(line[len("traffic-record: "):])
    if not rec or rec.get("sources_sha256") != sources_digest():
        return None
    if rec.get("batch") != batch or rec.get("launch", {}).get("bwd_chunk_mul") != launch["bwd_chunk_mul"]:
        return None
    if rec.get("launch", {}).get("bwd_pack", 0) != launch.get("bwd_pack", 0):
        return None
    return rec["hbm_bytes_per_launch"]


def profile_pass(B, steps=2):
    """`steps` forward + backward steps of the benchmark batch, then a 256 MiB device copy (the
    reference for the FETCH_SIZE / WRITE_SIZE scale); run under rocprofv3.  The big kernels run
    ~12% slower in the first steps of a fresh process than from about the eighth step on, where the
    bench's timed replays run, so a trace for durations takes ~10 steps and reads the last ones."""
    import numpy as np
    import torch
    import synth
    from paper_2505_22718_amd.plan import Plan, device_inputs
    wl = synth.make_workload("cfg1_batch", batch=B)
    plan = Plan.for_workload(wl)
    inp = device_inputs(wl, "cuda:0")
    out = torch.empty((B, plan.max_ell, plan.n_pairs), dtype=torch.float32, device="cuda:0")
    dC = torch.as_tensor(np.random.default_rng(0).standard_normal(out.shape), dtype=torch.float32, device="cuda:0")
    f64 = dict(dtype=torch.float64, device="cuda:0")
    grads = {"pk": torch.empty((B, len(wl["k"])), **f64), "bias": torch.empty((B, plan.max_tracers), **f64),
             "nz": torch.empty((B, plan.max_tracers, len(wl["z_nz"])), **f64),
             "D": torch.empty((B, len(wl["z_geom"])), **f64)}
    for _ in range(steps):
        plan.cl(inp, out)
        plan.backward_into(inp, dC, grads, reuse_forward=True)
    torch.cuda.synchronize()
    print(f"profile pass launch: batch {B}, {steps} steps, {json.dumps(plan.launch_config())}", flush=True)
    src = torch.ones(64 * 1024 * 1024, dtype=torch.float32, device="cuda:0")
    dst = torch.empty_like(src)
    dst.copy_(src)
    torch.cuda.synchronize()
    print("profile pass done: 2 steps, then a 268435456-byte copy", flush=True)


def profile_kgrowth_pass(B):
    """Two calls of scale-dependent growth on the benchmark batch (D(k, z) at 200 k nodes); run
    under rocprofv3."""
    import torch
    import synth
    from paper_2505_22718_amd.plan import Plan, device_inputs
    wl = synth.scale_dependent_growth(synth.make_workload("cfg1_batch", batch=B), 200)
    plan = Plan.for_workload(wl, n_interp=200)
    inp = device_inputs(wl, "cuda:0")
    D = torch.as_tensor(wl["D_kz"], dtype=torch.float64, device="cuda:0")
    for _ in range(2):
        plan.cl_kgrowth(inp, D)
    torch.cuda.synchronize()
    print("kgrowth profile pass done: 2 calls", flush=True)


def progress(msg):
    """One line on stderr per finished stage (the JSON line alone goes to stdout)."""
    print(f"bench: {msg}", file=sys.stderr, flush=True)


def profile_split_pass(B):
    """Two forward + backward steps of the 30-tracer split-precision batch (465 spectra x 200 l,
    N_k = N_chi = 2048; the adjoint through the workspace), then a 256 MiB device copy (the
    FETCH_SIZE / WRITE_SIZE reference); run under rocprofv3."""
    import numpy as np
    import torch
    import synth
    from paper_2505_22718_amd.plan import Plan, device_inputs
    wl = synth.make_workload("cfg4", batch=B)
    plan = Plan.for_workload(wl, precision="split_bf16")
    inp = device_inputs(wl, "cuda:0")
    C = torch.empty((B, plan.max_ell, plan.n_pairs), dtype=torch.float32, device="cuda:0")
    dC = torch.as_tensor(np.random.default_rng(0).standard_normal(tuple(C.shape)), dtype=torch.float32, device="cuda:0")
    for _ in range(2):
        plan.cl(inp, C)
        plan.backward(inp, dC, reuse_forward=True)
    torch.cuda.synchronize()
    src = torch.ones(64 * 1024 * 1024, dtype=torch.float32, device="cuda:0")
    dst = torch.empty_like(src)
    dst.copy_(src)
    torch.cuda.synchronize()
    print(f"split profile pass done: 2 steps of {B} points, then a 268435456-byte copy", flush=True)


def profile_ragged_pass(B, steps=2):
    """Forward + backward steps of the ragged batch (B points of 6, 10 or 15 tracers and 50..103
    multipoles) in launch shapes the autotuner picks for it in the bench (per-slot forward, the
    packed adjoint at two times the base multipole chunks); run under rocprofv3."""
    import numpy as np
    import torch
    import synth
    from paper_2505_22718_amd.plan import Plan, device_inputs
    wl = synth.make_workload("cfg3", batch=B)
    plan = Plan.for_workload(wl)
    plan.set_launch(fwd_mode=0, bwd_chunk_mul=2, bwd_pack=1)
    inp = device_inputs(wl, "cuda:0")
    C = torch.empty((B, plan.max_ell, plan.n_pairs), dtype=torch.float32, device="cuda:0")
    dC = torch.as_tensor(np.random.default_rng(0).standard_normal(tuple(C.shape)), dtype=torch.float32, device="cuda:0")
    for _ in range(steps):
        plan.cl(inp, C)
        plan.backward(inp, dC, reuse_forward=True)
    torch.cuda.synchronize()
    print(f"ragged profile pass done: {steps} steps of {B} points", flush=True)


def time_ms(fn, steps, stream):
    """Average device time of fn() over `steps` calls (HIP events on `stream`), after one warm-up."""
    import torch
    fn()
    torch.cuda.synchronize()
    start = torch.cuda.Event(enable_timing=True)
    end = torch.cuda.Event(enable_timing=True)
    start.record(stream)
    for _ in range(steps):
        fn()
    end.record(stream)
    torch.cuda.synchronize()
    return start.elapsed_time(end) / steps


def capture(fn):
    """fn() captured in a HIP graph (torch.cuda.CUDAGraph), after two eager calls on the capture's side
    stream.  The library's calls launch kernels only (no allocation, no memset), so they capture."""
    import gc
    import torch
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        for _ in range(2):
            fn()
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda.synchronize()
    gc.collect()  # nothing may be freed while the capture runs
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        fn()
    torch.cuda.synchronize()
    return g


def graph_ms(g, steps, warmup, stream):
    """Mean device time of `steps` replays after `warmup` (HIP events around the whole region)."""
    import torch
    for _ in range(warmup):
        g.replay()
    torch.cuda.synchronize()
    start = torch.cuda.Event(enable_timing=True)
    end = torch.cuda.Event(enable_timing=True)
    start.record(stream)
    for _ in range(steps):
        g.replay()
    end.record(stream)
    torch.cuda.synchronize()
    return start.elapsed_time(end) / steps


def graph_median_ms(g, n, stream):
    """Median device time of n replays, each between its own pair of HIP events."""
    import numpy as np
    import torch
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(n)]
    for a, b in ev:
        a.record(stream)
        g.replay()
        b.record(stream)
    torch.cuda.synchronize()
    return float(np.median([a.elapsed_time(b) for a, b in ev]))


def split_error(wl, C_gpu, points=(0,), ell_step=20):
    """Q12 error (|dC^{ij}| / sqrt(C^{ii} C^{jj})) of the GPU C_l against the FP64 oracle on whole
    points of the workload at every ell_step-th multipole: the maximum, and the maximum per multipole."""
    import numpy as np
    from oracle import fftlog
    sub = dict(wl)
    sub["ell_idx"] = np.ascontiguousarray(wl["ell_idx"][:, ::ell_step])
    sub["n_ell"] = np.full(wl["batch"], sub["ell_idx"].shape[1], np.int32)
    per_ell = None
    for b in points:
        C = fftlog.cl(sub, b)
        T = int(wl["n_tracers"][b])
        iu = np.triu_indices(T)
        g = C_gpu[b, ::ell_step][:, :C.shape[1]]
        diag = {int(i): C[:, p] for p, (i, j) in enumerate(zip(*iu)) if i == j}
        e = np.zeros(C.shape[0])
        for p, (i, j) in enumerate(zip(*iu)):
            e = np.maximum(e, np.abs(g[:, p] - C[:, p]) / np.sqrt(diag[int(i)] * diag[int(j)]))
        per_ell = e if per_ell is None else np.maximum(per_ell, e)
    return float(per_ell.max()), per_ell


def extra_configs(steps):
    """The other measured shapes: one point (latency), the ragged batch (256 points of 6, 10 or 15
    tracers and 50..103 multipoles), the 30-tracer split-precision batch (64 points, 465
    spectra x 200 l, N_k = N_chi = 2048; forward, and forward + the FP32 adjoint through the
    workspace) and
    scale-dependent growth (the benchmark batch with D(k, z) at 200 k nodes, forward only) and the
    Limber limit of the benchmark batch."""
    import numpy as np
    import torch
    import synth
    from paper_2505_22718_amd.plan import Plan, device_inputs
    out = {}
    stream = torch.cuda.current_stream()
    f64 = dict(dtype=torch.float64, device="cuda:0")

    def fwd_bwd(wl, precision=None, backward=True, tune=False):
        """Forward (and forward + backward): the median of 200 captured-graph replays, and the mean of
        eager calls beside it."""
        plan = Plan.for_workload(wl, precision=precision)
        inp = device_inputs(wl, "cuda:0")
        B = int(wl["batch"])
        C = torch.empty((B, plan.max_ell, plan.n_pairs), dtype=plan.out_dtype, device="cuda:0")
        dC = torch.as_tensor(np.random.default_rng(0).standard_normal(tuple(C.shape)), dtype=plan.out_dtype,
                             device="cuda:0")
        if tune:
            plan.autotune(inp, dC if backward else None)
        r = {"forward_ms_eager": time_ms(lambda: plan.cl(inp, C), steps, stream)}
        gf = capture(lambda: plan.cl(inp, C))
        graph_ms(gf, 20, 0, stream)
        r["forward_ms"] = graph_median_ms(gf, 200, stream)
        del gf
        if backward:
            g = {"pk": torch.empty((B, len(wl["k"])), **f64), "bias": torch.empty((B, plan.max_tracers), **f64),
                 "nz": torch.empty((B, plan.max_tracers, len(wl["z_nz"])), **f64),
                 "D": torch.empty((B, len(wl["z_geom"])), **f64)}

            def step():
                plan.cl(inp, C)
                plan.backward_into(inp, dC, g, reuse_forward=True)
            r["fwd_bwd_ms_eager"] = time_ms(step, steps, stream)
            gb = capture(step)
            graph_ms(gb, 20, 0, stream)
            r["fwd_bwd_ms"] = graph_median_ms(gb, 200, stream)
            del gb
        r["timing"] = "median of 200 captured-graph replays after 20 (eager means beside)"
        r["launch"] = plan.launch_config()
        return r, B, C

    r, B, _ = fwd_bwd(synth.make_workload("cfg1"))
    progress("one point timed")
    out["one_point_latency"] = dict(r, workload="1 point, 15 tracers x 103 l, N_k = N_chi = 1024, FP32")
    wl3 = synth.make_workload("cfg3")
    r, B, _ = fwd_bwd(wl3, tune=True)
    # algorithmic flops of the windows + projection over the ragged batch (each point its own T and L)
    f3 = sum(fused_kernel_flops(int(T), int(L), 1, wl3["n_chi"], len(wl3["k"]))
             for T, L in zip(wl3["n_tracers"], wl3["n_ell"]))
    out["ragged_batch"] = dict(r, points_per_s_fwd_bwd=B / (r["fwd_bwd_ms"] * 1e-3),
                               points_per_s_forward=B / (r["forward_ms"] * 1e-3),
                               roofline={"bound": "alu", "scope": "whole forward call (assembly, coefficients, "
                                         "windows + projection) against the windows' algorithmic flops",
                                         "achieved": f3 / (r["forward_ms"] * 1e-3) / 1e12,
                                         "peak": PEAK_FP32_VECTOR_TFLOPS, "unit": "TFLOP/s",
                                         "frac": f3 / (r["forward_ms"] * 1e-3) / 1e12 / PEAK_FP32_VECTOR_TFLOPS},
                               workload="256 points of 6/10/15 tracers and 50..103 l, FP32, autotuned launch")
    progress("ragged batch timed")
    wl4 = synth.make_workload("cfg4")
    r, B, C4 = fwd_bwd(wl4, precision="split_bf16")
    progress("30-tracer split batch timed; its error against the oracle next")
    f4 = fused_kernel_flops(30, 200, B, wl4["n_chi"], len(wl4["k"]))
    err, per_ell = split_error(wl4, C4.cpu().numpy().astype(np.float64))
    out["split_bf16_30_tracers"] = dict(
        r, points_per_s_forward=B / (r["forward_ms"] * 1e-3), points_per_s_fwd_bwd=B / (r["fwd_bwd_ms"] * 1e-3),
        max_rel_err_vs_oracle=err,
        rel_err_per_sampled_ell=[float(x) for x in per_ell],
        err_sample="point 0, all 465 spectra at every 20th of the 200 multipoles, FP64 FFTLog oracle, "
                   "|dC^{ij}| / sqrt(C^{ii} C^{jj})",
        roofline={"bound": "alu", "scope": "whole forward call against the windows' algorithmic flops",
                  "achieved": f4 / (r["forward_ms"] * 1e-3) / 1e12, "peak": PEAK_FP32_VECTOR_TFLOPS,
                  "unit": "TFLOP/s", "frac": f4 / (r["forward_ms"] * 1e-3) / 1e12 / PEAK_FP32_VECTOR_TFLOPS},
        workload="64 points x 30 tracers (465 spectra) x 200 l, N_k = N_chi = 2048, BF16 hi+lo projection, "
                 "FP32 adjoint")
    del C4
    progress("30-tracer split batch error done")
    # scale-dependent growth D(k, z) at the paper's default of 200 k nodes (swiftcl_cl_kgrowth)
    wl = synth.scale_dependent_growth(synth.make_workload("cfg1_batch", batch=256), 200)
    plan = Plan.for_workload(wl, n_interp=200)
    inp = device_inputs(wl, "cuda:0")
    D = torch.as_tensor(wl["D_kz"], **f64)
    C = torch.empty((256, plan.max_ell, plan.n_pairs), dtype=plan.out_dtype, device="cuda:0")
    ms = time_ms(lambda: plan.cl_kgrowth(inp, D, C), steps, stream)
    # the windows product: [103 l] x [chi nodes of the support] x [N_k] per tracer
    step = np.log(wl["k"][-1] / wl["k"][0]) / (len(wl["k"]) - 1)
    nodes = np.floor(np.log(wl["chi_z"][:, -1] / wl["chi_z"][:, 0]) / step) + 1.0
    gemm_flop = 2.0 * 103 * float(nodes.sum()) * len(wl["k"]) * 15
    progress("scale-dependent growth timed")
    out["scale_dependent_growth"] = dict(
        forward_ms=ms, points_per_s_forward=256 / (ms * 1e-3), windows_product_tflop=gemm_flop / 1e12,
        whole_call_tflops=gemm_flop / (ms * 1e-3) / 1e12, device_flags=plan.device_flags(),
        workload="256 points x 15 tracers x 103 l, N_k = N_chi = 1024, D(k, z) at 200 k nodes, FP32")
    del plan, D, C
    # the Limber limit of the benchmark batch on the same chi nodes (swiftcl_cl_limber)
    wl = synth.make_workload("cfg1_batch", batch=256)
    plan = Plan.for_workload(wl)
    inp = device_inputs(wl, "cuda:0")
    C = torch.empty((256, plan.max_ell, plan.n_pairs), dtype=plan.out_dtype, device="cuda:0")
    ms = time_ms(lambda: plan.cl_limber(inp, C), steps, stream)
    out["limber"] = dict(forward_ms=ms, points_per_s_forward=256 / (ms * 1e-3),
                         workload="256 points x 15 tracers x 103 l, Limber on the N_chi = 1024 nodes, FP32")
    return out


def cpu_baseline(wl, seconds, plan_out):
    """Time the FP64 oracle on as many points as fit in `seconds` (at least one)."""
    import numpy as np
    from oracle import fftlog
    try:
        from threadpoolctl import threadpool_info
        cores = max([i.get("num_threads", 1) for i in threadpool_info()] + [1])
    except Exception:
        cores = 1
    m = fftlog.method_for(wl)
    t0 = time.perf_counter()
    n = 0
    errs = []
    while True:
        C = fftlog.cl(wl, n, m)
        # GPU error of this point against the oracle: |dC^{ij}| / sqrt(C^{ii} C^{jj})
        T = int(wl["n_tracers"][n])
        iu = np.triu_indices(T)
        diag = {int(i): C[:, p] for p, (i, j) in enumerate(zip(*iu)) if i == j}
        g = plan_out[n][: C.shape[0], : C.shape[1]]
        for p, (i, j) in enumerate(zip(*iu)):
            errs.append(float(np.max(np.abs(g[:, p] - C[:, p]) / np.sqrt(diag[int(i)] * diag[int(j)]))))
        n += 1
        if time.perf_counter() - t0 >= seconds or n >= wl["batch"]:
            break
    dt = time.perf_counter() - t0
    model = "unknown CPU"
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    return {"value": n / dt, "unit": "sets/s", "cores": int(cores), "kind": "oracle",
            "cpu_model": model, "host_cpus": os.cpu_count(),
            "sample": f"{n} point(s) of the benchmark batch, full 120 spectra x 103 l each, "
                      f"FP64 FFTLog oracle (NumPy/SciPy, {int(cores)} BLAS threads on {model}), {dt:.1f} s"}, max(errs)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--batch", type=int, default=256)
    ap.add_argument("--cpu-seconds", type=float, default=15.0)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-extras", action="store_true", help="skip the one-point, ragged and split-precision lines")
    ap.add_argument("--profile-pass", action="store_true",
                    help="run two steps and a 256 MiB copy for rocprofv3 counters; no JSON line")
    ap.add_argument("--profile-steps", type=int, default=2, help="forward + backward steps of --profile-pass and --profile-ragged")
    ap.add_argument("--profile-kgrowth", action="store_true",
                    help="run two scale-dependent-growth calls of the batch for rocprofv3; no JSON line")
    ap.add_argument("--profile-split", action="store_true",
                    help="run two forward + backward steps of the 64-point, 30-tracer split-precision batch for rocprofv3; no JSON line")
    ap.add_argument("--profile-ragged", action="store_true",
                    help="run two forward + backward steps of the 256-point ragged batch for rocprofv3; no JSON line")
    args = ap.parse_args()
    world = int(os.environ.get("WORLD_SIZE", "1"))
    if args.gpus != 1 or world != 1:
        print("bench.py: the benchmark runs on one GPU only; a multi-GPU run is not supported "
              "(points would shard across GPUs with no exchange).", file=sys.stderr)
        sys.exit(2)

    if args.profile_pass:
        profile_pass(args.batch, args.profile_steps)
        return
    if args.profile_kgrowth:
        profile_kgrowth_pass(args.batch)
        return
    if args.profile_split:
        profile_split_pass(64)
        return
    if args.profile_ragged:
        profile_ragged_pass(256, args.profile_steps)
        return

    import numpy as np
    import torch

    import synth
    from paper_2505_22718_amd.plan import Plan, device_inputs

    B = args.batch
    wl = synth.make_workload("cfg1_batch", batch=B)
    plan = Plan.for_workload(wl)
    inp = device_inputs(wl, "cuda:0")
    out = torch.empty((B, plan.max_ell, plan.n_pairs), dtype=torch.float32, device="cuda:0")
    stream = torch.cuda.current_stream()

    rng = np.random.default_rng(0)
    dC = torch.as_tensor(rng.standard_normal((B, plan.max_ell, plan.n_pairs)), dtype=torch.float32,
                         device="cuda:0")
    f64 = dict(dtype=torch.float64, device="cuda:0")
    grads = {"pk": torch.empty((B, len(wl["k"])), **f64), "bias": torch.empty((B, plan.max_tracers), **f64),
             "nz": torch.empty((B, plan.max_tracers, len(wl["z_nz"])), **f64),
             "D": torch.empty((B, len(wl["z_geom"])), **f64)}

    # launch shapes picked by the library's autotuner on this batch (outside the timed region)
    tune_report = plan.autotune(inp, dC)
    progress("autotuned: " + tune_report)

    def step():
        plan.cl(inp, out)
        # the backward keeps the forward's assembly and FFTLog state (same inputs)
        plan.backward_into(inp, dC, grads, reuse_forward=True)

    # eager calls (the mean of K after W), for reference
    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    ms_eager = time_ms(step, args.steps, stream)
    ms_fwd_eager = time_ms(lambda: plan.cl(inp, out), args.steps, stream)
    # the timed steps: one step captured in a HIP graph, W warm-up replays, then K replays between two
    # HIP events (value); the median of 200 individually timed replays beside it
    g_step = capture(step)
    ms = graph_ms(g_step, args.steps, args.warmup, stream)
    ms_med = graph_median_ms(g_step, 200, stream)
    del g_step
    g_fwd = capture(lambda: plan.cl(inp, out))
    ms_fwd = graph_ms(g_fwd, args.steps, args.warmup, stream)
    ms_fwd_med = graph_median_ms(g_fwd, 200, stream)
    del g_fwd
    flags = plan.device_flags()
    progress(f"headline timed: {ms:.4f} ms per step ({B / (ms * 1e-3):.0f} sets/s)")

    fstages = np.mean([plan.cl_timed(inp, out) for _ in range(args.steps)], axis=0)
    bstages = np.mean([plan.backward_timed(inp, dC, grads, reuse_forward=True) for _ in range(args.steps)], axis=0)
    T, L, N, nk = 15, int(wl["n_ell"][0]), wl["n_chi"], len(wl["k"])
    kernels = {"k_windows_cl (windows + projection)": (float(fstages[2]), fused_kernel_flops(T, L, B, N, nk)),
               "k_bwd_windows (recompute + G W + adjoint FFTs)": (float(bstages[2]), bwd_kernel_flops(T, L, B, N, nk))}
    name = max(kernels, key=lambda k: kernels[k][0])
    kms, flops = kernels[name]
    achieved = flops / (kms * 1e-3) / 1e12
    traffic = traffic_bytes(B, plan.launch_config()) if name.startswith("k_bwd_windows") else None
    roofline = {"bound": "alu", "kernel": name, "achieved": achieved, "peak": PEAK_FP32_VECTOR_TFLOPS,
                "unit": "TFLOP/s", "frac": achieved / PEAK_FP32_VECTOR_TFLOPS, "traffic": traffic,
                "flops_per_launch": flops, "kernel_ms": kms}
    # both windows kernels against each roofline: FP32 VALU, the projection's MFMA share, HBM
    detail = {}
    for kname, (kt, kf) in kernels.items():
        tb = traffic_bytes(B, plan.launch_config()) if kname.startswith("k_bwd") else fwd_traffic_bytes(B, plan.launch_config())
        d = {"kernel_ms": kt, "alu_tflops": kf / (kt * 1e-3) / 1e12,
             "alu_frac": kf / (kt * 1e-3) / 1e12 / PEAK_FP32_VECTOR_TFLOPS,
             "hbm_bytes_per_launch": tb,
             "hbm_GBps": None if tb is None else tb / (kt * 1e-3) / 1e9,
             "hbm_frac": None if tb is None else tb / (kt * 1e-3) / 1e9 / PEAK_HBM_GBPS}
        if kname.startswith("k_windows_cl"):
            ca, ci = contraction_flops(T, L, B, nk)
            d.update(mfma_tflops_algorithmic=ca / (kt * 1e-3) / 1e12, mfma_tflops_issued=ci / (kt * 1e-3) / 1e12,
                     mfma_frac_issued=ci / (kt * 1e-3) / 1e12 / PEAK_FP32_MFMA_TFLOPS)
        detail[kname.split(" ")[0]] = d
    detail["note"] = ("alu: algorithmic flops over the whole kernel time against the FP32 vector peak; mfma: the "
                      "projection's flops (T(T+1) n_k per point and multipole algorithmic, the 16 x 16 Gram tile "
                      "issued) over the same time against the FP32 MFMA peak; hbm: bytes from the committed "
                      "rocprofv3 counter record (null when the kernel changed since) against 8 TB/s")

    result = {
        "metric": "C_\u2113 sets/s (15 tracers,103 \u2113) fwd & fwd+bwd at \u22641e-3 rel err vs FP64",
        "value": B / (ms * 1e-3),
        "forward_sets_per_s": B / (ms_fwd * 1e-3),
        "forward_ms_per_step": ms_fwd,
        "timing": "K replays of the step captured in a HIP graph after W warm-up replays (HIP events around "
                  "the K); the median of 200 individually timed replays and the mean of K eager calls beside",
        "ms_per_step_median200": ms_med,
        "forward_ms_per_step_median200": ms_fwd_med,
        "ms_per_step_eager": ms_eager,
        "forward_ms_per_step_eager": ms_fwd_eager,
        "unit": "sets/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": f"{B} points x (10 clustering + 5 lensing bins, 103 l in [2,2000], "
                               f"N_k = N_chi = 1024), per-point cosmology", "batch": B, "tracers": T,
                   "multipoles": L, "n_k": nk, "n_chi": N, "pass": "forward + backward (dP, db, dn(z), dD)"},
        "stage_ms": {"fwd_assembly": float(fstages[0]), "fwd_fftlog_coeffs": float(fstages[1]),
                     "fwd_windows_projection": float(fstages[2]), "bwd_assembly": float(bstages[0]),
                     "bwd_fftlog_coeffs": float(bstages[1]), "bwd_windows": float(bstages[2]),
                     "bwd_coeffs": float(bstages[3]), "bwd_geometry": float(bstages[4])},
        "device_flags": flags,
        "roofline_detail": detail,
        "launch": dict(plan.launch_config(), autotune=tune_report),
        "roofline": roofline,
    }
    if not args.no_extras:
        result["other_shapes"] = extra_configs(max(3, args.steps // 4))
    if not args.no_cpu_baseline:
        progress("oracle baseline")
        gpu_out = out.cpu().numpy().astype(np.float64)
        cb, err = cpu_baseline(wl, args.cpu_seconds, gpu_out)
        result["cpu_baseline"] = cb
        result["max_rel_err_vs_oracle"] = err
    print(json.dumps(result), flush=True)


if __name__ == "__main__":
    main()
