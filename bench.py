#!/usr/bin/env python3
"""Throughput of the fused V-trace loss+grad step on one MI355X.

One step is one vtrace_loss_grad call over a whole [T, B] batch: both
log-softmaxes, the importance weights, the reverse V-trace recursion, the
advantages, the three losses and the gradients w.r.t. logits and values.
Inputs are generated once, uploaded, and stay resident in HBM; the timed region
holds K back-to-back calls.  Prints one JSON line on stdout.

Default workload: the stress batch, T=1000, B=16384, A=18, fp32 logits,
rho_bar = c_bar = lambda = 1 (3.87 GB of algorithmic traffic per step, far
beyond the 256 MB Infinity Cache, so no cache flush is needed between steps).

``--head`` times vtrace_head_loss_grad instead: the learner's output layer
(hidden size 256, bfloat16) fused with the same V-trace step and the gradients
through the layer, on the stress shape drawn on the device.
"""

from __future__ import annotations

import argparse
import hashlib
import json
import math
import os
import platform
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_HBM_GBS = 8000.0  # MI355X HBM3E, AMD's published peak
METRIC = "trajectory steps/sec (T*B) for fused V-trace loss+grad; achieved HBM GB/s"
COUNTERS_FILE = os.path.join(ROOT, "profiles", "loss_grad_stress_counters.json")
HEAD_COUNTERS_FILE = os.path.join(ROOT, "profiles", "head_stress_counters.json")
# The sources each counted kernel is built from.
PLAIN_SOURCES = ("tiled.hip", "tiled_long_f32.hip", "tiled_impl.hpp", "row_stats.hpp", "device_common.hpp",
                 "wave_ops.hpp", "launch.hpp")
HEAD_SOURCES = ("head.hip", "head_impl.hpp", "head_h256.hip", "head.hpp", "device_common.hpp", "wave_ops.hpp",
                "launch.hpp")


def parse_args():
    ap = argparse.ArgumentParser(description=__doc__.split("\n")[0])
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=100)
    # The first few tens of milliseconds of calls after the upload run up to
    # 20% slower (measured: the first 5 of 30 calls 0.90 ms, the last 5
    # 0.74 ms), so the default warm-up covers them.
    ap.add_argument("--warmup", type=int, default=50)
    ap.add_argument("--config", type=int, default=4, help="synthetic workload id (0-4)")
    ap.add_argument("--params", type=int, default=0, help="parameter set of the workload")
    ap.add_argument("--bf16", action="store_true", help="bfloat16 logits")
    ap.add_argument("--kernel", choices=["auto", "lane_serial", "tiled", "tiled_single", "tiled_short",
                                         "tiled_short_single", "wide"],
                    default="auto",
                    help="force one V-trace kernel (where it applies); tiled_single keeps the tiled "
                         "kernel to one workgroup per tile, tiled_short to its 16-step tiles")
    ap.add_argument("--correction", choices=["vtrace", "none", "epsilon", "one_step_is"],
                    default="vtrace")
    ap.add_argument("--log-probs", action="store_true",
                    help="pass log mu(a_t|x_t) [T,B] instead of mu's logits")
    ap.add_argument("--grad-bf16", action="store_true", help="bfloat16 d_logits")
    ap.add_argument("--reward-transform", choices=["clip", "asymmetric"], default=None)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-seconds", type=float, default=12.0,
                    help="approximate CPU time for the oracle baseline sample")
    ap.add_argument("--cold", action="store_true",
                    help="write a 512 MB buffer before each timed call (outside its events) so "
                         "that no input is left in the 256 MB Infinity Cache; for workloads "
                         "smaller than the cache")
    ap.add_argument("--head", action="store_true",
                    help="time the fused output layer + V-trace call (stress shape, H=256)")
    ap.add_argument("--calibrate-copy", type=int, default=0, metavar="MIB",
                    help="only run plain device-to-device copies of MIB MiB (the reference "
                         "kernel for scaling HBM byte counters), then exit")
    return ap.parse_args()


def calibrate_copy(mib, reps):
    """Plain copies of a known size: what a byte counter reads for them calibrates
    the counter (bytes counted per byte moved)."""
    import torch
    n = mib * (1 << 20) // 4
    src = torch.ones(n, dtype=torch.float32, device="cuda")
    dst = torch.empty_like(src)
    dst.copy_(src)
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(reps):
        dst.copy_(src)
    e1.record()
    torch.cuda.synchronize()
    copy_ms = e0.elapsed_time(e1) / reps
    # a pure read for comparison: a sum over the same buffer
    src.sum()
    e0.record()
    for _ in range(reps):
        src.sum()
    e1.record()
    torch.cuda.synchronize()
    read_ms = e0.elapsed_time(e1) / reps
    # two reads and one write per element: the traffic mix of the V-trace step
    other = torch.ones_like(src)
    torch.add(src, other, out=dst)
    e0.record()
    for _ in range(reps):
        torch.add(src, other, out=dst)
    e1.record()
    torch.cuda.synchronize()
    mix_ms = e0.elapsed_time(e1) / reps
    print(json.dumps({"calibrate_copy_bytes_read": n * 4, "calibrate_copy_bytes_written": n * 4,
                      "copies": reps + 1, "copy_ms": copy_ms,
                      "copy_GBps_read_plus_write": 2 * n * 4 / copy_ms / 1e6,
                      "sum_read_GBps": n * 4 / read_ms / 1e6,
                      "add_2read_1write_GBps": 3 * n * 4 / mix_ms / 1e6}), flush=True)


def code_tokens(text: str) -> str:
    """C++ source with comments removed and whitespace runs collapsed: what the
    compiler sees, so that editing a comment keeps stored counters valid."""
    out, i, n = [], 0, len(text)
    while i < n:
        c = text[i]
        if text.startswith("//", i):
            j = text.find("\n", i)
            i = n if j < 0 else j
        elif text.startswith("/*", i):
            j = text.find("*/", i + 2)
            i = n if j < 0 else j + 2
            out.append(" ")
        elif c in "\"'":
            j = i + 1
            while j < n and text[j] != c:
                j += 2 if text[j] == "\\" else 1
            out.append(text[i:j + 1])
            i = j + 1
        else:
            out.append(c)
            i += 1
    return " ".join("".join(out).split())


def kernel_source_digest(files=PLAIN_SOURCES) -> str:
    """Hash of the code (comments and layout aside) of the HIP sources a kernel
    is built from, to tell whether stored counters still describe it."""
    csrc = os.path.join(ROOT, "paper_1802_01561_amd", "csrc")
    h = hashlib.sha256()
    for f in sorted(files):
        h.update(f.encode())
        with open(os.path.join(csrc, f), encoding="utf-8") as fh:
            h.update(code_tokens(fh.read()).encode())
    return h.hexdigest()[:16]


def algorithmic_bytes(T, B, A, logit_bytes, log_probs=False, grad_bytes=4, uses_mu=True):
    """Bytes one call must move: the target logit row, the behaviour logit row
    (or one log-probability; nothing for variants that ignore mu), action,
    reward, discount and value in; d_logits and d_values out; plus the
    bootstrap values."""
    behaviour = 0 if not uses_mu else (4 if log_probs else A * logit_bytes)
    per_step = A * logit_bytes + behaviour + 16 + A * grad_bytes + 4
    return T * B * per_step + 4 * B, per_step


def to_device(tr, torch, np):
    zt, yt = tr.logits_for_device()
    if tr.dtype == "bf16":
        z = torch.from_numpy(zt.view(np.int16)).view(torch.bfloat16)
        y = torch.from_numpy(yt.view(np.int16)).view(torch.bfloat16)
    else:
        z, y = torch.from_numpy(zt), torch.from_numpy(yt)
    d = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    return dict(target_logits=z.cuda(), behaviour_logits=y.cuda(), actions=d(tr.actions),
                rewards=d(tr.rewards), discounts=d(tr.discounts), values=d(tr.values),
                bootstrap_value=d(tr.bootstrap_value))


def stored_traffic(avg_kernel_ms, path=COUNTERS_FILE, files=PLAIN_SOURCES):
    """Counted HBM traffic of one launch, from committed rocprofv3 FETCH_SIZE and
    WRITE_SIZE runs scaled by the same counters' readings for a plain copy of
    known size, as (GB/s over this run's average launch time, bytes per launch).
    None when the counters are missing or were taken on other kernel sources."""
    try:
        with open(path) as fh:
            c = json.load(fh)
    except (OSError, ValueError):
        return None, None
    if c.get("kernel_source_digest") != kernel_source_digest(files):
        return None, None
    nbytes = c["hbm_bytes_per_launch"]
    return nbytes / (avg_kernel_ms * 1e-3) / 1e9, nbytes


def one_thread():
    """Context in which NumPy's BLAS and OpenMP pools use one thread, so that the
    oracle's timing is single-threaded whatever the host's defaults."""
    from threadpoolctl import threadpool_limits
    return threadpool_limits(limits=1)


def host_info():
    return {"cpu_model": cpu_model(), "host_cpus": os.cpu_count(),
            "host_cpus_available": len(os.sched_getaffinity(0)), "oracle_threads": 1}


def cpu_baseline(tr, p, target_s):
    """The fp64 oracle, as it stands, on a bounded sample of lanes (all T), on one
    host thread.  Lanes are independent, so the sample is run in chunks of at
    most 2048 lanes to bound host memory; the reported time is their sum."""
    import numpy as np
    import oracle
    from synth import subset_lanes

    def run(n):
        with one_thread():
            return run_threads(n)

    def run_threads(n):
        wall = 0.0
        for l0 in range(0, n, 2048):
            sub = subset_lanes(tr, np.arange(l0, min(n, l0 + 2048)))
            t0 = time.perf_counter()
            oracle.loss_and_grads(sub.target_logits, sub.behaviour_logits, sub.actions,
                                  sub.rewards, sub.discounts, sub.values, sub.bootstrap_value,
                                  p.rho_bar, p.c_bar, p.lam, p.baseline_cost, p.entropy_cost)
            wall += time.perf_counter() - t0
        return wall

    # Grow the sample until it costs a noticeable share of the target, then
    # scale it to about target_s.
    n = min(tr.B, 64)
    t = run(n)
    while t < target_s / 16 and n < tr.B:
        n = min(tr.B, n * 4)
        t = run(n)
    n = int(min(tr.B, max(n, n * target_s / max(t, 1e-6))))
    wall = run(n)
    return {
        "value": tr.T * n / wall,
        "unit": "steps/s",
        "cores": 1,
        "kind": "oracle",
        "sample": f"{n} of {tr.B} lanes x all T={tr.T} steps ({tr.T * n} steps) of the same "
                  f"batch, fp64 NumPy oracle, one thread, {wall:.1f} s wall",
        **host_info(),
    }


def cpu_model():
    name = platform.processor()
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return name


def timed_calls(step, K, W, stream, flush=None):
    """W untimed calls, then K calls bracketed by synchronisations, each between
    two HIP events on the launch stream (``flush``, when given, runs before
    each call, outside its events).  Returns (per-call event ms, wall ms per
    call)."""
    import numpy as np
    import torch
    for _ in range(W):
        step()
    torch.cuda.synchronize()
    starts = [torch.cuda.Event(enable_timing=True) for _ in range(K)]
    ends = [torch.cuda.Event(enable_timing=True) for _ in range(K)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(K):
        if flush is not None:
            flush()
        starts[i].record(stream)
        step()
        ends[i].record(stream)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    return np.array([s.elapsed_time(e) for s, e in zip(starts, ends)]), (t1 - t0) * 1e3 / K


def head_algorithmic_bytes(T, B, A, H, grad_bytes, log_probs=False):
    """Bytes the fused output-layer call must move: per step the hidden row
    (bfloat16), the behaviour logit row (or log mu(a_t|x_t)), action, reward and
    discount in and the d_hidden row out; per call the bootstrap values, the
    layer's parameters in and their gradients out."""
    per_step = 2 * H + (4 if log_probs else 4 * A) + 12 + grad_bytes * H
    per_call = 4 * B + (2 * H * (A + 1) + 4 * (A + 1)) + (4 * H * (A + 1) + 4 * (A + 1) + 16)
    return T * B * per_step + per_call, per_step


def head_cpu_baseline(d, p, target_s, T, B):
    """The fp64 oracle of the fused call, as it stands, on a bounded sample of
    lanes (all T) copied back from the device, one host thread."""
    import numpy as np
    import oracle
    from synth import head_batch_from_device

    def run(n):
        wall = 0.0
        for l0 in range(0, n, 256):
            hb = head_batch_from_device(d, list(range(l0, min(n, l0 + 256))))
            with one_thread():
                t0 = time.perf_counter()
                oracle.head_loss_and_grads(hb.hidden, hb.weight, hb.bias, hb.behaviour_logits,
                                           hb.actions, hb.rewards, hb.discounts,
                                           hb.bootstrap_value, p.rho_bar, p.c_bar, p.lam,
                                           p.baseline_cost, p.entropy_cost)
                wall += time.perf_counter() - t0
        return wall

    n = 16
    t = run(n)
    while t < target_s / 16 and n < B:
        n = min(B, n * 4)
        t = run(n)
    n = int(min(B, max(n, n * target_s / max(t, 1e-6))))
    wall = run(n)
    return {
        "value": T * n / wall,
        "unit": "steps/s",
        "cores": 1,
        "kind": "oracle",
        "sample": f"{n} of {B} lanes x all T={T} steps ({T * n} steps) of the same batch, "
                  f"fp64 NumPy oracle of the output layer + V-trace (BLAS on one thread), "
                  f"{wall:.1f} s wall",
        **host_info(),
    }


def run_head(args):
    """The fused output layer + V-trace call on the stress shape with H = 256."""
    import numpy as np
    import torch

    import paper_1802_01561_amd as vt
    from synth import HEAD_WORKLOADS, SEED_BASE, Params, make_head_device

    c = HEAD_WORKLOADS["stress"]
    T, B, A, H = c["T"], c["B"], c["A"], c["H"]
    seed = SEED_BASE + 1004
    p = Params()
    t_gen = time.perf_counter()
    d = make_head_device(T, B, A, H, seed, "cuda")
    torch.cuda.synchronize()
    print(f"[bench] head stress T={T} B={B} A={A} H={H} {p.label()} "
          f"(generated on the device in {time.perf_counter() - t_gen:.1f} s)", file=sys.stderr,
          flush=True)
    grad_dtype = torch.bfloat16 if args.grad_bf16 else torch.float32
    beh, behaviour = d["behaviour_logits"], "logits"
    if args.log_probs:
        # log mu(a_t|x_t), computed once on the device outside the timed region
        lp = torch.log_softmax(beh, dim=-1)
        beh = lp.gather(-1, d["actions"].long()[..., None])[..., 0].contiguous()
        del lp
        behaviour = "log_probs"
    ws = vt.Workspace(T, B, A, H=H)
    f32 = dict(dtype=torch.float32, device="cuda")
    out = vt.HeadLossGrad(torch.empty(4, **f32), torch.empty((T, B, H), dtype=grad_dtype, device="cuda"),
                          torch.empty((H, A + 1), **f32), torch.empty(A + 1, **f32),
                          None, None, None, None)
    stream = torch.cuda.current_stream()

    def step():
        vt.vtrace_head_loss_grad(d["hidden"], d["weight"], d["bias"], beh,
                                 d["actions"], d["rewards"], d["discounts"], d["bootstrap_value"],
                                 p.rho_bar, p.c_bar, p.lam, p.baseline_cost, p.entropy_cost,
                                 workspace=ws, out=out, grad_dtype=grad_dtype, behaviour=behaviour)

    call_ms, ms_per_step = timed_calls(step, args.steps, args.warmup, stream)
    avg_ms = float(call_ms.mean())
    grad_bytes = 2 if args.grad_bf16 else 4
    alg_bytes, per_step = head_algorithmic_bytes(T, B, A, H, grad_bytes, args.log_probs)
    achieved = alg_bytes / (avg_ms * 1e-3) / 1e9
    mfma_flop = 3 * 2 * T * B * H * (A + 1)  # forward, d_hidden, d_weight
    print(f"[bench] head call avg {avg_ms:.4f} ms (min {call_ms.min():.4f}); wall "
          f"{ms_per_step:.4f} ms/step; {achieved:.1f} GB/s algorithmic; "
          f"{mfma_flop / (avg_ms * 1e-3) / 1e12:.1f} TFLOP/s of matrix products; losses "
          f"{out.losses.cpu().tolist()}", file=sys.stderr, flush=True)
    counted = not args.grad_bf16 and not args.log_probs
    traffic, traffic_bytes = (stored_traffic(avg_ms, HEAD_COUNTERS_FILE, HEAD_SOURCES) if counted
                              else (None, None))
    result = {
        "metric": METRIC,
        "value": T * B / (ms_per_step * 1e-3),
        "unit": "steps/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16-mfma/f32",
        "data": "synthetic",
        "config": {
            "workload": f"stress + output layer: T={T} B={B} A={A} H={H}, bf16 hidden and "
                        f"weights, f32 behaviour {'log-probabilities' if args.log_probs else 'logits'}, "
                        f"{'bf16' if args.grad_bf16 else 'f32'} "
                        f"d_hidden, rho_bar=c_bar=lambda=1",
            "T": T, "B": B, "A": A, "H": H, "seed": seed,
        },
        "kernel_ms_avg": avg_ms,
        "kernel_ms_median": float(np.median(call_ms)),
        "kernel_ms_min": float(call_ms.min()),
        "timing": "back-to-back calls; value from the wall clock of the timed region",
        "alg_bytes_per_launch": alg_bytes,
        "alg_bytes_per_step": per_step,
        "traffic_bytes_per_launch": traffic_bytes,
        "mfma_tflops": mfma_flop / (avg_ms * 1e-3) / 1e12,
        "roofline": {
            "bound": "hbm",
            "achieved": achieved,
            "peak": PEAK_HBM_GBS,
            "unit": "GB/s",
            "frac": achieved / PEAK_HBM_GBS,
            "traffic": traffic,
        },
    }
    if not args.no_cpu_baseline:
        result["cpu_baseline"] = head_cpu_baseline(d, p, args.cpu_seconds, T, B)
    print(json.dumps(result), flush=True)


def main():
    args = parse_args()
    if args.gpus != 1:
        print("bench.py measures one GPU only: the library has no multi-GPU path. Lanes are "
              "independent, so the batch axis would shard across GPUs with no communication "
              "except a 4-float loss all-reduce.", file=sys.stderr)
        sys.exit(2)
    if args.calibrate_copy:
        calibrate_copy(args.calibrate_copy, max(1, args.steps))
        return
    if args.kernel != "auto":
        os.environ["VTRACE_KERNEL"] = args.kernel
    if args.head:
        import torch
        if not torch.cuda.is_available():
            print("bench.py needs a GPU", file=sys.stderr)
            sys.exit(1)
        torch.cuda.set_device(0)
        run_head(args)
        return

    import numpy as np
    import torch

    import paper_1802_01561_amd as vt
    from synth import PARAM_SETS, WORKLOADS, make_config

    if not torch.cuda.is_available():
        print("bench.py needs a GPU", file=sys.stderr)
        sys.exit(1)
    torch.cuda.set_device(0)

    t_gen = time.perf_counter()
    tr = make_config(args.config, bf16=args.bf16)
    p = PARAM_SETS[args.config][args.params]
    dev = to_device(tr, torch, np)
    T, B, A = tr.T, tr.B, tr.A
    behaviour = "logits"
    if args.log_probs:
        # log mu(a_t|x_t), computed once on the device outside the timed region
        lp = torch.log_softmax(dev["behaviour_logits"].float(), dim=-1)
        dev["behaviour_logits"] = lp.gather(-1, dev["actions"].long()[..., None])[..., 0].contiguous()
        del lp
        behaviour = "log_probs"
    grad_dtype = torch.bfloat16 if args.grad_bf16 else torch.float32
    print(f"[bench] {tr.name} T={T} B={B} A={A} {tr.dtype} {p.label()} "
          f"(generated+uploaded in {time.perf_counter() - t_gen:.1f} s)", file=sys.stderr, flush=True)

    ws = vt.Workspace(T, B, A)
    f32 = dict(dtype=torch.float32, device="cuda")
    out = vt.LossGrad(torch.empty(4, **f32), torch.empty((T, B, A), dtype=grad_dtype, device="cuda"),
                      torch.empty((T, B), **f32), None, None, None)
    stream = torch.cuda.current_stream()

    def step():
        vt.vtrace_loss_grad(**dev, rho_bar=p.rho_bar, c_bar=p.c_bar, lam=p.lam,
                            baseline_cost=p.baseline_cost, entropy_cost=p.entropy_cost,
                            workspace=ws, out=out, correction=args.correction, behaviour=behaviour,
                            reward_transform=args.reward_transform, grad_dtype=grad_dtype)

    K = args.steps
    flush = None
    if args.cold:
        flush_buf = torch.empty(512 << 20, dtype=torch.uint8, device="cuda")
        flush = lambda: flush_buf.fill_(1)  # noqa: E731
    kernel_ms, ms_per_step = timed_calls(step, K, args.warmup, stream, flush)
    main_losses = out.losses.clone()  # on the stream: the sets below reuse `out`
    is_counted_workload = (WORKLOADS[args.config]["name"] == "stress" and args.params == 0
                           and not args.bf16 and args.kernel == "auto" and args.correction == "vtrace"
                           and not args.log_probs and not args.grad_bf16
                           and args.reward_transform is None)
    # The stress batch's other parameter sets on the same inputs, timed right
    # after the main region (fewer calls each, as many warm-up calls): every
    # set is held to the same tolerance and takes the same kernel.
    other_sets = []
    if is_counted_workload and len(PARAM_SETS[args.config]) > 1:
        for q in PARAM_SETS[args.config][1:]:
            def step_q(q=q):
                vt.vtrace_loss_grad(**dev, rho_bar=q.rho_bar, c_bar=q.c_bar, lam=q.lam,
                                    baseline_cost=q.baseline_cost, entropy_cost=q.entropy_cost,
                                    workspace=ws, out=out, grad_dtype=grad_dtype)
            q_ms, _ = timed_calls(step_q, max(20, K // 5), args.warmup, stream, None)
            other_sets.append((q, q_ms))
    if args.cold:
        # the wall clock includes the flushes: the cold rate comes from the
        # events around each call alone
        ms_per_step = float(np.median(kernel_ms))
    steps_per_s = T * B / (ms_per_step * 1e-3)
    logit_bytes = 2 if args.bf16 else 4
    alg_bytes, per_step = algorithmic_bytes(T, B, A, logit_bytes, args.log_probs,
                                            2 if args.grad_bf16 else 4,
                                            args.correction in ("vtrace", "one_step_is"))
    avg_kernel_ms = float(kernel_ms.mean())
    achieved = alg_bytes / (avg_kernel_ms * 1e-3) / 1e9
    losses = main_losses.cpu().tolist()
    print(f"[bench] kernel avg {avg_kernel_ms:.4f} ms (min {kernel_ms.min():.4f}, median "
          f"{np.median(kernel_ms):.4f}); wall {ms_per_step:.4f} ms/step; {achieved:.1f} GB/s "
          f"algorithmic; losses {losses}", file=sys.stderr, flush=True)

    traffic, traffic_bytes = stored_traffic(avg_kernel_ms) if is_counted_workload else (None, None)
    result = {
        "metric": METRIC,
        "value": steps_per_s,
        "unit": "steps/s",
        "n_gpus": 1,
        "steps": K,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16-in/f32" if args.bf16 else "f32",
        "data": "synthetic",
        "config": {
            "workload": f"{tr.name}: T={T} B={B} A={A} {tr.dtype} logits, "
                        f"rho_bar={p.rho_bar} c_bar={p.c_bar} lambda={p.lam}"
                        + (f", correction={args.correction}" if args.correction != "vtrace" else "")
                        + (", behaviour log-probs" if args.log_probs else "")
                        + (", bf16 d_logits" if args.grad_bf16 else "")
                        + (f", rewards {args.reward_transform}" if args.reward_transform else ""),
            "T": T, "B": B, "A": A, "logits": tr.dtype,
            "rho_bar": p.rho_bar if math.isfinite(p.rho_bar) else "inf",
            "c_bar": p.c_bar if math.isfinite(p.c_bar) else "inf",
            "lambda": p.lam, "baseline_cost": p.baseline_cost, "entropy_cost": p.entropy_cost,
            "seed": tr.seed,
        },
        "kernel_ms_avg": avg_kernel_ms,
        "kernel_ms_median": float(np.median(kernel_ms)),
        "timing": ("cold: a 512 MB buffer is written before each call; value from the median "
                   "event time of the calls" if args.cold else
                   "back-to-back calls; value from the wall clock of the timed region"),
        "alg_bytes_per_launch": alg_bytes,
        "traffic_bytes_per_launch": traffic_bytes,
        "kernel_ms_min": float(kernel_ms.min()),
        "alg_bytes_per_step": per_step,
        "roofline": {
            "bound": "hbm",
            "achieved": achieved,
            "peak": PEAK_HBM_GBS,
            "unit": "GB/s",
            "frac": achieved / PEAK_HBM_GBS,
            "traffic": traffic,
        },
    }
    if other_sets:
        result["other_param_sets"] = [
            {"rho_bar": q.rho_bar if math.isfinite(q.rho_bar) else "inf",
             "c_bar": q.c_bar if math.isfinite(q.c_bar) else "inf", "lambda": q.lam,
             "calls": int(q_ms.size), "kernel_ms_avg": float(q_ms.mean()),
             "frac": alg_bytes / (float(q_ms.mean()) * 1e-3) / 1e9 / PEAK_HBM_GBS}
            for q, q_ms in other_sets]
    if not args.no_cpu_baseline:
        result["cpu_baseline"] = cpu_baseline(tr, p, args.cpu_seconds)
    print(json.dumps(result), flush=True)


if __name__ == "__main__":
    main()
