"""Benchmark of the GRPO/PPO trainer-step core on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload 7b|1.5b|longcot|lossonly|tiny]

One step is one pass of the whole hot path over one synthetic batch that is
already resident in HBM: group advantages, then rft_ppo_clip_step - per-token
log-probs and entropy through the lm_head (online log-sum-exp, logits kept only
for one chunk of rows), the PPO-clip/KL loss, and the backward to the hidden
states and the lm_head weight (the loss-only workload: log-softmax statistics,
loss and d_logits from given logits in one fused call).  Prints one JSON line.

The default run (the 7B-shape step) also frees that batch and times the
loss-only workload (``lossonly``: its HBM fraction), and measures two ceilings
on the same device (``ceilings``): a device copy moving the loss-only call's
read and write bytes, and the best rate of the vendor bf16 GEMM (hipBLASLt
through torch) on large shapes of the step's GEMMs.
"""
from __future__ import annotations

import argparse
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "response tokens/s for fused logprob+PPO-clip fwd+bwd; % bf16 MFMA / HBM peak"
PEAK_BF16_TFLOPS = 2500.0
PEAK_HBM_GBS = 8000.0
WORKLOADS = {"tiny": 0, "1.5b": 1, "7b": 2, "longcot": 3, "lossonly": 4}

# HBM bytes per launch of the dominant kernel from rocprofv3 FETCH_SIZE and
# WRITE_SIZE (one run each), scaled by what the same counters read for a plain
# copy of known size (read x2.0, write x1.0).  Valid only for the kernel
# sources they were taken with: a changed source reports null.
TRAFFIC = {
    # forward GEMM alone (k_gemm384<EPI_STATS> on the tile-blocked copies, one launch over
    # all valid rows)
    "7b": {"sources": {'k_gemm_mfma.hip': '0cc59ef48596356f', 'rft_internal.h': 'a778fbc47a9f52d0'},
           "bytes": 172748926.9 * 1024 * 2.0 + 1174430.6 * 1024 * 1.0},
    # every kernel of one rft_ppo_clip_step call and its advantages (24 dispatches, two
    # row chunks)
    "step_7b": {"sources": {'k_gemm_mfma.hip': '0cc59ef48596356f', 'k_step.hip': 'a920d8a6385f4246', 'k_layout.hip': '59fafc69e9c8b096', 'k_adv_loss.hip': '20f27cec6e4001a4', 'k_tokens.hip': '2e004762720e0e21', 'tokens_device.h': 'd5c28753c1c6f594', 'rft_internal.h': 'a778fbc47a9f52d0', 'rft_abi.hip': '0a71af3bbc7c6fe8'},
                "bytes": 616371101.2 * 1024 * 2.0 + 164158424.2 * 1024 * 1.0},
    "lossonly": {"sources": {'k_logits.hip': '4ea4f0a25bbfcd3f', 'rft_internal.h': 'a778fbc47a9f52d0'},
                 "bytes": 8758803.0 * 1024 * 2.0 + 19480261.2 * 1024 * 1.0},
}


def traffic_gb(workload):
    import hashlib
    t = TRAFFIC.get(workload)
    if t is None:
        return None
    csrc = os.path.join(ROOT, "paper_2505_17826_amd", "csrc")
    for f, h in t["sources"].items():
        with open(os.path.join(csrc, f), "rb") as fh:
            if hashlib.sha256(fh.read()).hexdigest()[:16] != h:
                return None
    return t["bytes"] / 1e9


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--workload", default="7b", choices=sorted(WORKLOADS))
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-seconds", type=float, default=15.0,
                    help="target CPU time of the oracle baseline sample")
    ap.add_argument("--ws-gb", type=float, default=0.0,
                    help="workspace of the fused step in GB (default 0: the library's "
                         "recommended size); the step takes the largest row chunk that fits, "
                         "so a smaller workspace means more, smaller chunks")
    ap.add_argument("--ws-one-chunk", action="store_true",
                    help="size the workspace so that one row chunk holds the batch's valid "
                         "rows (rft_workspace_bytes_rows)")
    ap.add_argument("--copy-probe", type=float, default=0.0, metavar="GB",
                    help="only run a plain device copy of GB gigabytes (the known-size kernel "
                         "that scales the HBM byte counters) and exit")
    return ap.parse_args()


def copy_probe(gb):
    """A plain fp32 device-to-device copy of a known size, three launches."""
    import torch
    n = int(gb * 1e9) // 4
    x = torch.ones(n, dtype=torch.float32, device="cuda")
    y = torch.empty_like(x)
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(3):
        y.copy_(x)
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / 3
    print(json.dumps({"copy_probe_bytes_each_way": n * 4, "ms_per_copy": ms,
                      "GB_per_s_read_plus_write": 2 * n * 4 / ms / 1e6}), flush=True)


def _stats_ms(xs):
    import numpy as np
    a = np.asarray(xs, dtype=np.float64)
    return {"median": float(np.median(a)), "mean": float(a.mean()), "min": float(a.min()),
            "max": float(a.max())}


def source_rev():
    """git revision of the tree when .git is there, and a hash of the sources
    that the measured path runs (the library sources, the header, this file),
    which identifies the code also where the tree was copied without .git."""
    import hashlib
    import subprocess
    rev = None
    try:
        r = subprocess.run(["git", "-C", ROOT, "rev-parse", "--short=12", "HEAD"],
                           capture_output=True, text=True, timeout=10)
        if r.returncode == 0:
            rev = r.stdout.strip()
            d = subprocess.run(["git", "-C", ROOT, "status", "--porcelain", "--untracked-files=no"],
                               capture_output=True, text=True, timeout=10)
            if d.returncode == 0 and d.stdout.strip():
                rev += "-dirty"
    except Exception:
        rev = None
    h = hashlib.sha256()
    csrc = os.path.join(ROOT, "paper_2505_17826_amd", "csrc")
    for f in sorted(os.listdir(csrc)) + ["../../include/rft.h", "../../bench.py"]:
        with open(os.path.join(csrc, f), "rb") as fh:
            h.update(f.encode() + fh.read())
    return {"git_rev": rev, "source_sha16": h.hexdigest()[:16]}


def _time_events(fn, reps):
    import torch
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
          for _ in range(reps)]
    for a, z in ev:
        a.record()
        fn()
        z.record()
    torch.cuda.synchronize()
    return [a.elapsed_time(z) for a, z in ev]


def measure_ceilings(read_gb, write_gb, reps=5):
    """Ceilings measured on this device.

    copy_mix: a device copy of read_gb gigabytes (read once, written once) plus
    a fill of the remaining write_gb - read_gb gigabytes (written only), the
    byte mix of the loss-only call (every valid row read once, every row of
    d_logits written once); rate = (read_gb + write_gb) / (copy + fill time),
    best of torch's copy and an elementwise copy kernel.
    gemm_bf16: hipBLASLt (torch.matmul, bf16 in, fp32 accumulate) on the
    shapes of the step's forward (M x V-slab x d) and d_hidden (M x d x V-slab)
    GEMMs, best of the two, against the 2.5 PFLOP/s bf16 peak."""
    import torch
    out = {}
    n_rd = int(read_gb * 1e9) // 4
    n_fill = max(0, int((write_gb - read_gb) * 1e9) // 4)
    x = torch.randn(n_rd, device="cuda")
    y = torch.empty_like(x)
    f = torch.empty(max(n_fill, 1), device="cuda")
    for fn in (lambda: y.copy_(x), lambda: torch.mul(x, 1.0, out=y), lambda: f.zero_()):
        fn()
    torch.cuda.synchronize()
    best = None
    for name, cp in (("torch copy_", lambda: y.copy_(x)),
                     ("elementwise mul by 1", lambda: torch.mul(x, 1.0, out=y))):
        t_cp = _stats_ms(_time_events(cp, reps))["median"]
        t_fill = _stats_ms(_time_events(lambda: f.zero_(), reps))["median"] if n_fill else 0.0
        gbs = (read_gb + write_gb) / ((t_cp + t_fill) / 1e3)
        if best is None or gbs > best["GB_per_s"]:
            best = {"GB_per_s": gbs, "frac_of_peak": gbs / PEAK_HBM_GBS, "kernel": name,
                    "copy_ms": t_cp, "fill_ms": t_fill, "read_GB": read_gb, "write_GB": write_gb}
    out["copy_mix"] = best
    del x, y, f
    torch.cuda.empty_cache()
    gemms = []
    for (M, Nn, K, what) in ((32768, 19008, 3584, "forward-like: rows x V/8 x d"),
                             (32768, 3584, 38016, "d_hidden-like: rows x d x V/4")):
        a = torch.randn(M, K, device="cuda").to(torch.bfloat16)
        bT = torch.randn(Nn, K, device="cuda").to(torch.bfloat16)
        mm = lambda: torch.matmul(a, bT.t())
        mm()
        torch.cuda.synchronize()
        ms = _stats_ms(_time_events(mm, reps))["median"]
        tf = 2.0 * M * Nn * K / (ms / 1e3) / 1e12
        gemms.append({"shape": [M, Nn, K], "what": what, "ms": ms, "TFLOP_per_s": tf,
                      "frac_of_peak": tf / PEAK_BF16_TFLOPS})
        del a, bT
        torch.cuda.empty_cache()
    best_g = max(gemms, key=lambda g: g["TFLOP_per_s"])
    out["gemm_bf16"] = {"TFLOP_per_s": best_g["TFLOP_per_s"],
                        "frac_of_peak": best_g["frac_of_peak"],
                        "kernel": "hipBLASLt via torch.matmul (NT, bf16)", "shapes": gemms}
    return out


def measure_lossonly(R, synth, dev, steps, warmup):
    """The loss-only workload (fp32 logits [32768, 151936], 10% of rows masked):
    group advantages + rft_ppo_clip_fused_logits per step; per-call event
    times of the fused call, its algorithmic bytes and HBM fraction."""
    import numpy as np
    import torch
    cfg = synth.config(4)
    b = synth.make_batch(cfg, dev)
    tok = R.Tokens(b.seq_start, b.mask, b.ids)
    N = int(b.mask.sum().item())
    T, V = b.T, cfg.V
    params = R.ppo_params(cfg.eps_low, cfg.eps_high, cfg.beta, cfg.agg)
    f32 = dict(dtype=torch.float32, device=dev)
    adv = torch.empty(cfg.n_seq, **f32)
    logp, ent, lse, grad = (torch.empty(T, **f32) for _ in range(4))
    stats = torch.zeros(R.STATS_BYTES, dtype=torch.uint8, device=dev)
    dl = torch.empty_like(b.logits)
    ws = torch.empty(max(1, R.workspace_bytes(R.RFT_OP_PPO_FUSED_LOGITS, tok, 0, V)),
                     dtype=torch.uint8, device=dev)
    R.rft_token_logprobs_from_logits(tok, b.logits, logp=logp, entropy=ent, lse=lse)
    old = torch.where(b.mask.bool(), logp + b.old_noise, torch.zeros_like(logp))
    ref = torch.where(b.mask.bool(), logp + b.ref_noise, torch.zeros_like(logp))
    evs = []

    def step(ev=None):
        R.rft_group_advantages(b.rewards, cfg.group, out=adv)
        if ev is not None:
            ev[0].record()
        R.rft_ppo_clip_fused_logits(tok, b.logits, old, ref, adv, params, logp=logp, entropy=ent,
                                    lse=lse, grad_logp=grad, d_logits=dl, stats=stats, ws=ws)
        if ev is not None:
            ev[1].record()
    for _ in range(warmup):
        step()
    torch.cuda.synchronize()
    evs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
           for _ in range(steps)]
    for e in evs:
        step(e)
    torch.cuda.synchronize()
    call_ms = [a.elapsed_time(z) for a, z in evs]
    st = _stats_ms(call_ms)
    gb = (N * V * 4 + T * V * 4) / 1e9
    res = {"workload": cfg.name, "valid_tokens": N, "T": T, "V": V,
           "kernel": "k_logits_fused_cached (one workgroup per row: stats, loss, d_logits)",
           "calls": steps, "ms_per_call": st, "algorithmic_GB_per_call": gb,
           "GB_per_s": gb / (st["mean"] / 1e3), "GB_per_s_median": gb / (st["median"] / 1e3),
           "peak_GB_per_s": PEAK_HBM_GBS, "frac": gb / (st["mean"] / 1e3) / PEAK_HBM_GBS,
           "tokens_per_s": N / (st["median"] / 1e3),
           "traffic": traffic_gb("lossonly"), "traffic_unit": "GB per launch",
           "loss": R.stats_to_dict(stats)["loss"],
           "read_GB": N * V * 4 / 1e9, "write_GB": T * V * 4 / 1e9}
    del b, dl, ws
    torch.cuda.empty_cache()
    return res


def cpu_baseline(batch, target_s, extra):
    """Time the float64 oracle on a bounded sample of the same workload."""
    import numpy as np
    from oracle import rft_oracle as O
    try:
        from threadpoolctl import threadpool_info
        cores = max([i.get("num_threads", 1) for i in threadpool_info()] or [1])
    except Exception:  # pragma: no cover
        cores = os.cpu_count()
    cfg = batch.cfg
    mask = batch.mask.cpu().numpy()
    valid = np.nonzero(mask)[0]

    def run(n_rows):
        rows = valid[:n_rows]
        ss = np.array([0, n_rows], dtype=np.int32)
        m = np.ones(n_rows, dtype=np.uint8)
        ids = batch.ids.cpu().numpy()[rows]
        rewards = np.array([1.0], dtype=np.float64)
        # old / reference log-probs: a fixed offset from a plain value (the
        # oracle's cost does not depend on them); the timed call is one step
        old = np.full(n_rows, -np.log(cfg.V) + 0.1)
        ref = old - 0.2
        if cfg.dtype == "logits":
            z = batch.logits[rows].cpu()
            t0 = time.perf_counter()
            O.loss_only_step(z, ids, m, ss, rewards, 1, old, ref, cfg.eps_low, cfg.eps_high,
                             cfg.beta, cfg.agg)
        else:
            H = batch.H[rows].cpu()
            W = extra["W_cpu"]
            t0 = time.perf_counter()
            O.trainer_step(H, W, ids, m, ss, rewards, 1, old, ref, cfg.eps_low, cfg.eps_high,
                           cfg.beta, cfg.agg)
        return time.perf_counter() - t0

    if cfg.dtype != "logits":
        extra["W_cpu"] = batch.W.cpu()
    n, t = 32, 0.0
    run(n)                       # warm-up (first touches of the weight)
    t = run(n)
    # the per-call overhead makes small samples look slow: rescale until the
    # sample takes at least 60% of the target (or covers every valid token)
    for _ in range(3):
        if t >= 0.6 * target_s or n >= valid.size:
            break
        n = int(min(valid.size, max(n + 1, n * target_s / max(t, 1e-3))))
        t = run(n)
    return {"value": n / t, "unit": "tokens/s", "cores": int(cores), "kind": "oracle",
            "sample": f"first {n} valid tokens of the same batch as one rollout, whole step "
                      f"(log-probs, loss, dH and dW over the full vocabulary) in float64; "
                      f"{t:.1f} s"}


def main():
    args = parse()
    if args.copy_probe > 0:
        copy_probe(args.copy_probe)
        return
    if args.gpus != 1:
        print(f"bench.py: the library runs on one GPU only (asked for --gpus {args.gpus}); "
              "multi-GPU runs (sharding by whole GRPO groups) are not implemented",
              file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    import paper_2505_17826_amd as R
    from gen import synth

    assert torch.cuda.is_available(), "bench.py needs the GPU"
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    cid = WORKLOADS[args.workload]
    cfg = synth.config(cid)
    t_gen = time.perf_counter()
    b = synth.make_batch(cfg, dev)
    torch.cuda.synchronize()
    t_gen = time.perf_counter() - t_gen
    print(f"[bench] workload {cfg.name}: T={b.T} generated in {t_gen:.1f} s", file=sys.stderr,
          flush=True)

    tok = R.Tokens(b.seq_start, b.mask, b.ids)
    N = int(b.mask.sum().item())
    n_seq = cfg.n_seq
    params = R.ppo_params(cfg.eps_low, cfg.eps_high, cfg.beta, cfg.agg)
    T = b.T
    f32 = dict(dtype=torch.float32, device=dev)
    adv = torch.empty(n_seq, **f32)
    logp = torch.empty(T, **f32)
    ent = torch.empty(T, **f32)
    lse = torch.empty(T, **f32)
    grad = torch.empty(T, **f32)
    stats = torch.zeros(R.STATS_BYTES, dtype=torch.uint8, device=dev)
    V = cfg.V
    events = []

    if cfg.dtype == "logits":
        dl = torch.empty_like(b.logits)
        ws_f = torch.empty(max(1, R.workspace_bytes(R.RFT_OP_PPO_FUSED_LOGITS, tok, 0, V)),
                           dtype=torch.uint8, device=dev)
        # rollout-side log-probs for the old / reference policies (setup, untimed)
        R.rft_token_logprobs_from_logits(tok, b.logits, logp=logp, entropy=ent, lse=lse)
        old = torch.where(b.mask.bool(), logp + b.old_noise, torch.zeros_like(logp))
        ref = torch.where(b.mask.bool(), logp + b.ref_noise, torch.zeros_like(logp))

        def step(ev=None):
            R.rft_group_advantages(b.rewards, cfg.group, out=adv)
            if ev is not None:
                ev[0].record()
            R.rft_ppo_clip_fused_logits(tok, b.logits, old, ref, adv, params, logp=logp,
                                        entropy=ent, lse=lse, grad_logp=grad, d_logits=dl,
                                        stats=stats, ws=ws_f)
            if ev is not None:
                ev[1].record()
        dom_name = "k_logits_fused_cached (one workgroup per row: stats, loss, d_logits)"
        # algorithmic bytes: read every valid row once, write every row of d_logits once
        dom_work = (N * V * 4 + T * V * 4) / 1e9  # GB
        bound = "hbm"
    else:
        d = cfg.d
        dt = R.RFT_BF16 if cfg.dtype == "bf16" else R.RFT_F32
        dH = torch.empty((T, d), **f32)
        dW = torch.empty((V, d), **f32)
        ws_fwd = torch.empty(R.workspace_bytes(R.RFT_OP_TOKEN_LOGPROBS, tok, d, V, dt),
                             dtype=torch.uint8, device=dev)
        ws_step_bytes = R.workspace_bytes(R.RFT_OP_PPO_STEP, tok, d, V, dt)
        if args.ws_one_chunk:
            # N is known here, outside the timed region
            ws_step_bytes = R.workspace_bytes_rows(R.RFT_OP_PPO_STEP, tok, d, V, dt, max(N, 1))
        if args.ws_gb > 0:
            ws_step_bytes = int(args.ws_gb * 1e9)
        chunk_rows = R.chunk_rows(R.RFT_OP_PPO_STEP, tok, d, V, dt, ws_step_bytes)
        ws_step = torch.empty(ws_step_bytes, dtype=torch.uint8, device=dev)
        # rollout-side log-probs for the old / reference policies (setup, untimed)
        R.rft_token_logprobs(tok, b.H, b.W, logp=logp, entropy=ent, lse=lse, ws=ws_fwd)
        old = torch.where(b.mask.bool(), logp + b.old_noise, torch.zeros_like(logp))
        ref = torch.where(b.mask.bool(), logp + b.ref_noise, torch.zeros_like(logp))

        def step(ev=None):
            R.rft_group_advantages(b.rewards, cfg.group, out=adv)
            if ev is not None:
                ev[0].record()
            R.rft_ppo_clip_step(tok, b.H, b.W, old, ref, adv, params, logp=logp, entropy=ent,
                                lse=lse, grad_logp=grad, d_hidden=dH, d_weight=dW, stats=stats,
                                ws=ws_step)
            if ev is not None:
                ev[1].record()

        def fwd_kernel_ms(reps=3):
            """The forward GEMM with online log-sum-exp alone (rft_token_logprobs), timed
            after the benchmark: its per-launch rate is the kernel-level roofline."""
            e = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
                 for _ in range(reps)]
            for a, z in e:
                a.record()
                R.rft_token_logprobs(tok, b.H, b.W, logp=logp, entropy=ent, lse=lse, ws=ws_fwd)
                z.record()
            torch.cuda.synchronize()
            return float(np.mean([a.elapsed_time(z) for a, z in e]))
        dom_name = ("rft_ppo_clip_step: every MFMA GEMM of the step (forward with online LSE "
                    "and fp16 logit store, dH, dW) plus the dZ pass; 6*N*d*V algorithmic flops "
                    "per call")
        dom_work = 6.0 * N * d * V / 1e12  # TFLOP
        bound = "mfma" if cfg.dtype == "bf16" else "alu"

    torch.cuda.synchronize()
    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    # per step: one event pair around the whole step (advantages + the call)
    # and one around the call alone (the dominant launch sequence)
    sev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
           for _ in range(args.steps)]
    evs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
           for _ in range(args.steps)]
    t_start = torch.cuda.Event(enable_timing=True)
    t_end = torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    t_start.record()
    for k in range(args.steps):
        sev[k][0].record()
        step(evs[k])
        sev[k][1].record()
    t_end.record()
    torch.cuda.synchronize()
    ms_total = t_start.elapsed_time(t_end) / max(args.steps, 1)
    step_ms = _stats_ms([a.elapsed_time(z) for a, z in sev])
    ms = step_ms["median"]
    dom_ms = float(np.mean([a.elapsed_time(z) for a, z in evs])) if args.steps else float("nan")
    st = R.stats_to_dict(stats)
    tokens_per_s = N / (ms / 1e3)

    out = {
        "metric": METRIC, "value": tokens_per_s, "unit": "tokens/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": ms,
        "ms_per_step_stats": {**step_ms, "mean_over_timed_region": ms_total,
                              "note": "value and ms_per_step use the median step"},
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": {"bf16": "bf16", "f32": "f32", "logits": "f32"}[cfg.dtype],
        "data": "synthetic (seeded; shapes and distributions of the workload, no dataset)",
        "config": {"workload": cfg.name, "n_seq": n_seq, "group": cfg.group, "T": T,
                   "workspace_bytes": (ws_step_bytes if cfg.dtype != "logits" else None),
                   "chunk_rows": (chunk_rows if cfg.dtype != "logits" else None),
                   "valid_tokens": N, "V": V, "d": cfg.d, "eps": [cfg.eps_low, cfg.eps_high],
                   "kl_coef": cfg.beta, "agg": cfg.agg},
    }
    if bound == "hbm":
        ach = dom_work / (dom_ms / 1e3)
        out["roofline"] = {"bound": "hbm", "achieved": ach, "peak": PEAK_HBM_GBS, "unit": "GB/s",
                           "frac": ach / PEAK_HBM_GBS, "traffic": traffic_gb(args.workload),
                           "traffic_unit": "GB per launch", "kernel": dom_name,
                           "ms_per_launch": dom_ms}
    else:
        ach = dom_work / (dom_ms / 1e3)
        peak = PEAK_BF16_TFLOPS if bound == "mfma" else 157.3
        out["roofline"] = {"bound": bound, "achieved": ach, "peak": peak, "unit": "TFLOP/s",
                           "frac": ach / peak, "traffic": traffic_gb("step_" + args.workload),
                           "traffic_unit": "GB per launch", "kernel": dom_name,
                           "ms_per_launch": dom_ms}
        alg = 6.0 * N * cfg.d * V / 1e12
        out["step_mfma"] = {"algorithmic_tflop": alg, "algorithmic_tflops": alg / (ms / 1e3),
                            "frac_algorithmic": alg / (ms / 1e3) / peak,
                            "executed_flop_per_token": "6dV (logits formed once, not recomputed)"}
        fms = fwd_kernel_ms()
        fw = 2.0 * N * cfg.d * V / 1e12
        out["roofline_fwd_kernel"] = {
            "kernel": ("k_gemm384<EPI_STATS> on tile-blocked copies (recommended workspace) via "
                       "rft_token_logprobs: the whole call, timed after the benchmark"),
            "bound": bound, "achieved": fw / (fms / 1e3), "peak": peak, "unit": "TFLOP/s",
            "frac": fw / (fms / 1e3) / peak, "ms_per_launch": fms,
            "traffic": traffic_gb(args.workload), "traffic_unit": "GB per launch"}
    out["loss"] = st["loss"]
    out["clipfrac"] = st["clipfrac"]
    out["rev"] = source_rev()
    if cfg.dtype == "logits":
        lo_read, lo_write = N * V * 4 / 1e9, T * V * 4 / 1e9
    else:
        # the second target: the loss-only workload's HBM fraction, timed after
        # this workload's buffers are freed
        del dH, dW, ws_fwd, ws_step
        torch.cuda.empty_cache()
        print("[bench] loss-only workload", file=sys.stderr, flush=True)
        out["lossonly"] = measure_lossonly(R, synth, dev, max(args.steps, 5), args.warmup)
        lo_read, lo_write = out["lossonly"]["read_GB"], out["lossonly"]["write_GB"]
    print("[bench] ceilings", file=sys.stderr, flush=True)
    out["ceilings"] = measure_ceilings(lo_read, lo_write)
    if not args.no_cpu_baseline:
        print("[bench] timing the float64 oracle on a CPU sample", file=sys.stderr, flush=True)
        out["cpu_baseline"] = cpu_baseline(b, args.cpu_seconds, {})
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
