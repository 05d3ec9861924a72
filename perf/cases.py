"""Performance cases of the trainer-step core: what a fine-tuning loop calls, over its range.

A case is one call chain of a training program through the package's entry points:

  step        rft_group_advantages + rft_ppo_clip_step: the policy update of the head (forward,
              loss, d_hidden, d_weight) from hidden states, bf16 or fp32
  logprobs    rft_token_logprobs: the forward alone, as when a trainer recomputes the old or
              reference log-probs of a batch
  sft         rft_token_logprobs + rft_sft_loss_fwd + rft_ppo_clip_loss_bwd: supervised
              fine-tuning through the head with the separate forward and backward
  loss_logits rft_ppo_clip_fused_logits: the loss-only path from fp32 logits that exist
  dpo_logits  rft_token_logprobs_from_logits + rft_dpo_loss_fwd + rft_ppo_clip_loss_bwd_logits:
              preference training from logits
  loss        rft_group_advantages_ids + rft_ppo_clip_loss_fwd: advantages over explicit groups
              and the loss from given log-probs (the metrics of a whole batch, an update whose
              head runs elsewhere)

Layouts are padded [n_seq, pad] batches whose rollouts use a random part of their rows (the
rest is masked), or, with mask_frac, rows masked at random.  Workspaces, outputs and the
statistics buffer are made once and reused, as a training loop does.
"""
import math

import numpy as np
import torch

import paper_2505_17826_amd as R

DEV = "cuda"


def _step(name, **kw):
    c = dict(name=name, kind="step", dtype="bf16", prompts=1, group=8, lo=1, pad=16, d=64, V=512,
             agg=0, eps_high=0.2, beta=0.001, ent=0.0, mix=0.0)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: 32 rollouts of 8 tokens through a toy fp32 head; launches and host time
        _step("step_f32_tiny", dtype="f32", prompts=4, lo=8, pad=8, d=64, V=512, beta=0.01),
        # an fp32 head (no low-precision copy of the weights) on a small batch
        _step("step_f32_mid", dtype="f32", prompts=2, lo=32, pad=128, d=1024, V=32000),
        # one prompt's rollouts as a micro-batch through the 7B-shape head, MIX with one expert
        # rollout in eight
        _step("step_7b_micro", lo=128, pad=512, d=3584, V=152064, mix=0.1),
        # an ordinary batch through the 1.5B-shape head, entropy bonus, token-mean weights
        _step("step_1p5b_batch", prompts=8, lo=256, pad=1024, d=1536, V=151936, agg=1, ent=0.01),
        # the largest: 32 rollouts of up to 2048 tokens through the 7B-shape head
        _step("step_7b_large", prompts=4, lo=512, pad=2048, d=3584, V=152064),
        # recomputing the old log-probs (and the entropy) of a batch, 1.5B shape
        dict(name="logprobs_1p5b", kind="logprobs", dtype="bf16", n_seq=16, lo=128, pad=1024,
             d=1536, V=151936),
        # one SFT micro-batch through the 7B-shape head
        dict(name="sft_7b_micro", kind="sft", dtype="bf16", n_seq=4, lo=64, pad=512, d=3584,
             V=152064, agg=1),
        # the loss-only path on few rows: latency
        dict(name="loss_logits_few", kind="loss_logits", prompts=1, group=8, pad=16, V=151936,
             mask_frac=0.1, beta=0.01, ent=0.0, agg=0),
        # the loss-only path on a batch, 10% of the rows masked: HBM
        dict(name="loss_logits_batch", kind="loss_logits", prompts=32, group=8, pad=32, V=151936,
             mask_frac=0.1, beta=0.01, ent=0.0, agg=0),
        # an unpadded vocabulary (rows of logits not 16-byte aligned), with the entropy bonus
        dict(name="loss_logits_odd", kind="loss_logits", prompts=4, group=8, pad=64, V=50001,
             mask_frac=0.1, beta=0.01, ent=0.01, agg=1),
        # preference pairs from logits over a small vocabulary
        dict(name="dpo_logits", kind="dpo_logits", n_seq=16, lo=32, pad=256, V=32000),
        # advantages and loss of a whole 128-rollout batch from given log-probs
        dict(name="loss_given_logps", kind="loss", prompts=16, group=8, lo=512, pad=2048,
             V=152064, beta=0.001, agg=0, mix=0.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step_f32", "logprobs", "sft", "loss_logits", "loss_logits",
                       "dpo_logits", "loss"])
    if kind in ("step", "step_f32", "logprobs", "sft"):
        f32 = kind == "step_f32"
        V = _log(rng, 512, 50000) if f32 else _log(rng, 8000, 152064)
        d = _log(rng, 64, 1024) if f32 else 8 * _log(rng, 64, 448)
        pad = _log(rng, 8, 128) if f32 else _log(rng, 32, 2048)
        group = rng.choice([4, 8, 16])
        prompts = _log(rng, 1, 8)
        # no larger than the largest listed case of the kind
        cap = (2048 * 1024 * 32000 if f32 else 65536 * 3584 * 152064 if kind == "step"
               else 16384 * 1536 * 151936)
        rows = min(65536, max(16, cap // (d * V)))
        pad = max(2, min(pad, rows // (group * prompts)))
        lo = max(1, pad // rng.choice([1, 2, 4, 8]))
        if kind in ("step", "step_f32"):
            c = _step("", dtype="f32" if f32 else "bf16", prompts=prompts, group=group, lo=lo,
                      pad=pad, d=d, V=V, agg=rng.choice([0, 1]), eps_high=rng.choice([0.2, 0.28]),
                      ent=rng.choice([0.0, 0.01]), mix=rng.choice([0.0, 0.1]))
            c.pop("name")
            return c
        c = dict(kind=kind, dtype="bf16", n_seq=prompts * group, lo=lo, pad=pad, d=d, V=V)
        if kind == "sft":
            c["agg"] = rng.choice([0, 1])
        return c
    if kind == "loss":
        pad = _log(rng, 8, 2048)
        return dict(kind=kind, prompts=_log(rng, 1, 16), group=rng.choice([4, 8]),
                    lo=max(1, pad // 4), pad=pad, V=_log(rng, 512, 152064), beta=0.001,
                    agg=rng.choice([0, 1]), mix=rng.choice([0.0, 0.1]))
    V = _log(rng, 1000, 152064)
    rows = min(32768, 8192 * 151936 // V)
    if kind == "dpo_logits":
        n_seq = 2 * _log(rng, 1, 16)
        pad = max(2, min(_log(rng, 8, 1024), rows // (2 * n_seq)))
        return dict(kind=kind, n_seq=n_seq, lo=max(1, pad // 4), pad=pad, V=V)
    group, prompts = rng.choice([4, 8]), _log(rng, 1, 32)
    pad = max(1, min(_log(rng, 4, 1024), rows // (group * prompts)))
    return dict(kind=kind, prompts=prompts, group=group, pad=pad, V=V,
                mask_frac=rng.choice([0.0, 0.1, 0.5]), beta=0.01, ent=rng.choice([0.0, 0.01]),
                agg=rng.choice([0, 1]))


# ---------------------------------------------------------------------------- inputs --
def _n_seq(c):
    return c["n_seq"] if "n_seq" in c else c["prompts"] * c["group"]


def _layout(c, seed):
    """seq_start, mask on the host (numpy) of the case's padded batch."""
    r = np.random.default_rng([seed, 1])
    n, pad = _n_seq(c), c["pad"]
    start = (np.arange(n + 1, dtype=np.int64) * pad).astype(np.int32)
    if "mask_frac" in c:
        mask = np.ones(n * pad, np.uint8)
        mask[r.choice(n * pad, size=int(round(c["mask_frac"] * n * pad)), replace=False)] = 0
    else:
        lengths = r.integers(c["lo"], pad + 1, size=n)
        mask = (np.arange(pad)[None, :] < lengths[:, None]).astype(np.uint8).reshape(-1)
    return start, mask


def _rewards(c, seed):
    """0/1 rewards, each prompt with its own success rate; a prompt whose rollouts all agree has
    its first one flipped (trainers drop groups without a signal)."""
    r = np.random.default_rng([seed, 2])
    p = r.random((c["prompts"], 1))
    v = (r.random((c["prompts"], c["group"])) < p).astype(np.float32)
    same = (v == v[:, :1]).all(1)
    v[same, 0] = 1 - v[same, 0]
    return torch.from_numpy(v.reshape(-1)).to(DEV)


def _sample(z, g):
    """Ids drawn from softmax(z) (Gumbel-max) and their log-probs."""
    e = torch.empty_like(z).exponential_(generator=g)
    y = (z - e.log_()).argmax(1)
    return y, z.gather(1, y[:, None])[:, 0] - torch.logsumexp(z, 1)


def _old_ref(logp, valid, eps_low, eps_high, g):
    """Old and reference log-probs: the current ones plus noise of variance 0.05 / 0.1.  A token
    whose ratio lies within 0.002 of a clip bound is moved past that, so that rounding does not
    decide which branch it takes."""
    d = torch.randn(logp.shape, generator=g, device=DEV) * math.sqrt(0.05)  # logp - old
    for b in (math.log1p(-eps_low), math.log1p(eps_high)):
        d = torch.where((d - b).abs() < 2e-3, torch.full_like(d, b + 2e-3), d)
    old = logp - d
    ref = logp + torch.randn(logp.shape, generator=g, device=DEV) * math.sqrt(0.1)
    zero = torch.zeros_like(logp)
    return torch.where(valid, old, zero), torch.where(valid, ref, zero)


def _stats():
    """The statistics buffer and its values as a program reads them (n_clipped through clipfrac)."""
    buf = torch.zeros(R.STATS_BYTES, dtype=torch.uint8, device=DEV)
    f, i = buf.view(torch.float64), buf.view(torch.int64)
    return buf, {"means": f[0:7], "sft_loss": f[11:12], "entropy_loss": f[13:14],
                 "n_valid": i[7:9], "n_bad_ids": i[10:11], "n_expert": i[12:13]}


def _f32(*shape):
    return torch.empty(shape, dtype=torch.float32, device=DEV)


def _ws(nbytes):
    return torch.empty(max(16, nbytes), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    c, kind = case, case["kind"]
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    start, mask = _layout(c, seed)
    T, n_seq, V = mask.size, start.size - 1, c["V"]
    s = dict(case=c)
    start_d, mask_d = torch.from_numpy(start).to(DEV), torch.from_numpy(mask).to(DEV)
    valid = mask_d != 0
    rows = valid.nonzero()[:, 0]
    ids = torch.zeros(T, dtype=torch.int32, device=DEV)
    logp = torch.zeros(T, device=DEV)
    expert = None
    if c.get("mix"):
        expert = torch.zeros(n_seq, dtype=torch.uint8, device=DEV)
        expert[::8] = 1  # one rollout in eight is an expert's

    chunk = max(1, min(T, (1 << 29) // V))
    if kind in ("step", "logprobs", "sft"):
        d, dt = c["d"], torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
        code = R.RFT_BF16 if c["dtype"] == "bf16" else R.RFT_F32
        # unit-variance hidden states, logits of standard deviation 2
        H = torch.randn((T, d), generator=g, device=DEV, dtype=torch.float32).to(dt)
        H *= valid[:, None]
        W = (torch.randn((V, d), generator=g, device=DEV) * (2 / math.sqrt(d))).to(dt)
        for r0 in range(0, rows.numel(), chunk):
            rr = rows[r0:r0 + chunk]
            z = (H[rr] @ W.t()).float()
            y, lp = _sample(z, g)
            # the sampled logit in fp32 (the product above rounds it to the data type)
            zy = (H[rr].float() * W[y].float()).sum(1)
            ids[rr], logp[rr] = y.int(), lp + zy - z.gather(1, y[:, None])[:, 0]
            del z
        s.update(H=H, W=W)
    elif kind in ("loss_logits", "dpo_logits"):
        logits = torch.empty((T, V), device=DEV)
        for r0 in range(0, T, chunk):
            z = logits[r0:r0 + chunk]
            z.normal_(0.0, 2.0, generator=g)
            y, lp = _sample(z, g)
            ids[r0:r0 + chunk], logp[r0:r0 + chunk] = y.int(), lp
        ids *= valid
        logp *= valid
        s.update(logits=logits)
    else:
        ids = (torch.rand(T, generator=g, device=DEV) * V).int() * valid
        logp = -5.0 * torch.rand(T, generator=g, device=DEV) * valid
    tok = R.Tokens(start_d, mask_d, ids, expert)
    s.update(tok=tok, T=T)

    if kind in ("step", "loss_logits", "loss"):
        eh = c.get("eps_high", 0.2)
        s["old"], s["ref"] = _old_ref(logp, valid, 0.2, eh, g)
        s["params"] = R.ppo_params(0.2, eh, c["beta"], c["agg"], mix_mu=c.get("mix", 0.0),
                                   entropy_coef=c.get("ent", 0.0))
        s["rewards"], s["adv"] = _rewards(c, seed), _f32(n_seq)
    if kind in ("step", "loss_logits", "loss", "sft"):
        s["stats"], s["read"] = _stats()
    if kind == "step":
        s.update(logp=_f32(T), ent=_f32(T), lse=_f32(T), grad=_f32(T), dH=_f32(T, d), dW=_f32(V, d),
                 ws=_ws(R.workspace_bytes(R.RFT_OP_PPO_STEP, tok, d, V, code)))
    elif kind == "logprobs":
        s.update(logp=_f32(T), ent=_f32(T), lse=_f32(T),
                 ws=_ws(R.workspace_bytes(R.RFT_OP_TOKEN_LOGPROBS, tok, d, V, code)))
    elif kind == "sft":
        s.update(logp=_f32(T), ent=_f32(T), lse=_f32(T), grad=_f32(T), dH=_f32(T, d), dW=_f32(V, d),
                 ws=_ws(max(R.workspace_bytes(R.RFT_OP_TOKEN_LOGPROBS, tok, d, V, code),
                            R.workspace_bytes(R.RFT_OP_SFT_FWD, tok, 0, V),
                            R.workspace_bytes(R.RFT_OP_PPO_BWD, tok, d, V, code))))
    elif kind == "loss_logits":
        s.update(logp=_f32(T), ent=_f32(T), lse=_f32(T), grad=_f32(T), dz=_f32(T, V),
                 ws=_ws(R.workspace_bytes(R.RFT_OP_PPO_FUSED_LOGITS, tok, 0, V)))
        R.rft_group_advantages(s["rewards"], c["group"], out=s["adv"])
    elif kind == "dpo_logits":
        s["ref"] = (logp + torch.randn(T, generator=g, device=DEV) * math.sqrt(0.1)) * valid
        stats = torch.zeros(R.DPO_STATS_BYTES, dtype=torch.uint8, device=DEV)
        s.update(logp=_f32(T), ent=_f32(T), lse=_f32(T), grad=_f32(T), dz=_f32(T, V),
                 seq=_f32(n_seq), stats=stats,
                 read={"means": stats.view(torch.float64)[0:5], "counts": stats.view(torch.int64)[5:8]},
                 ws=_ws(R.workspace_bytes(R.RFT_OP_DPO_FWD, tok, 0, V)))
    else:
        # explicit groups: rollouts shuffled over the prompts, a few left out (lagged reward)
        r = np.random.default_rng([seed, 3])
        gid = r.permutation(np.repeat(np.arange(c["prompts"]), c["group"])).astype(np.int32)
        gid[r.random(n_seq) < 0.05] = -1
        s.update(gid=torch.from_numpy(gid).to(DEV), logp=logp, grad=_f32(T),
                 ent=(3.0 + torch.rand(T, generator=g, device=DEV)) * valid,
                 ws=_ws(R.workspace_bytes(R.RFT_OP_PPO_FWD, tok, 0, V)),
                 ws_adv=_ws(int(R.lib().rft_group_advantages_ids_workspace_bytes(n_seq, c["prompts"]))))
    return s


# ------------------------------------------------------------------------------ pass --
def run(s):
    c, tok = s["case"], s["tok"]
    kind = c["kind"]
    if kind == "step":
        R.rft_group_advantages(s["rewards"], c["group"], out=s["adv"])
        R.rft_ppo_clip_step(tok, s["H"], s["W"], s["old"], s["ref"], s["adv"], s["params"],
                            logp=s["logp"], entropy=s["ent"], lse=s["lse"], grad_logp=s["grad"],
                            d_hidden=s["dH"], d_weight=s["dW"], stats=s["stats"], ws=s["ws"])
        return {"adv": s["adv"], "logp": s["logp"], "entropy": s["ent"], "lse": s["lse"],
                "grad_logp": s["grad"], "d_hidden": s["dH"], "d_weight": s["dW"], "stats": s["read"]}
    if kind == "logprobs":
        R.rft_token_logprobs(tok, s["H"], s["W"], logp=s["logp"], entropy=s["ent"], lse=s["lse"],
                             ws=s["ws"])
        return {"logp": s["logp"], "entropy": s["ent"], "lse": s["lse"]}
    if kind == "sft":
        R.rft_token_logprobs(tok, s["H"], s["W"], logp=s["logp"], entropy=s["ent"], lse=s["lse"],
                             ws=s["ws"])
        R.rft_sft_loss_fwd(tok, c["V"], s["logp"], agg=c["agg"], grad_logp=s["grad"],
                           stats=s["stats"], ws=s["ws"])
        R.rft_ppo_clip_loss_bwd(tok, s["H"], s["W"], s["lse"], s["grad"], d_hidden=s["dH"],
                                d_weight=s["dW"], ws=s["ws"])
        return {"logp": s["logp"], "entropy": s["ent"], "lse": s["lse"], "grad_logp": s["grad"],
                "d_hidden": s["dH"], "d_weight": s["dW"], "stats": s["read"]}
    if kind == "loss_logits":
        R.rft_ppo_clip_fused_logits(tok, s["logits"], s["old"], s["ref"], s["adv"], s["params"],
                                    logp=s["logp"], entropy=s["ent"], lse=s["lse"],
                                    grad_logp=s["grad"], d_logits=s["dz"], stats=s["stats"],
                                    ws=s["ws"])
        return {"logp": s["logp"], "entropy": s["ent"], "lse": s["lse"], "grad_logp": s["grad"],
                "d_logits": s["dz"], "stats": s["read"]}
    if kind == "dpo_logits":
        R.rft_token_logprobs_from_logits(tok, s["logits"], logp=s["logp"], entropy=s["ent"],
                                         lse=s["lse"])
        R.rft_dpo_loss_fwd(tok, c["V"], s["logp"], s["ref"], beta=0.1, grad_logp=s["grad"],
                           seq_logp=s["seq"], stats=s["stats"], ws=s["ws"])
        R.rft_ppo_clip_loss_bwd_logits(tok, s["logits"], s["lse"], s["grad"], d_logits=s["dz"])
        return {"logp": s["logp"], "entropy": s["ent"], "lse": s["lse"], "grad_logp": s["grad"],
                "seq_logp": s["seq"], "d_logits": s["dz"], "stats": s["read"]}
    R.rft_group_advantages_ids(s["rewards"], s["gid"], c["prompts"], out=s["adv"], ws=s["ws_adv"])
    R.rft_ppo_clip_loss_fwd(tok, c["V"], s["logp"], s["old"], s["ref"], s["adv"], s["params"],
                            entropy=s["ent"], grad_logp=s["grad"], stats=s["stats"], ws=s["ws"])
    return {"adv": s["adv"], "grad_logp": s["grad"], "stats": s["read"]}


# ------------------------------------------------------------------------------ work --
def work(case):
    c, kind = case, case["kind"]
    T, V = _n_seq(c) * c["pad"], c["V"]
    # valid rows: the mean of the length distribution
    N = T * (1 - c["mask_frac"]) if "mask_frac" in c else _n_seq(c) * (c["lo"] + c["pad"]) / 2
    row = 5  # mask and token id
    if kind in ("step", "logprobs", "sft"):
        d, e = c["d"], 2 if c["dtype"] == "bf16" else 4
        nbytes = N * d * e + V * d * e + T * (row + 12)
        if kind == "logprobs":
            return {"bytes": nbytes, "flops": 2 * N * d * V}
        nbytes += T * d * 4 + V * d * 4 + T * (12 if kind == "step" else 4)
        return {"bytes": nbytes, "flops": 6 * N * d * V}
    if kind in ("loss_logits", "dpo_logits"):
        # each valid row read once and every row of the gradient written once
        return {"bytes": 4 * N * V + 4 * T * V + T * (row + 24), "flops": 8 * N * V}
    return {"bytes": T * (row + 20), "flops": 40 * N}


def tolerance(case):
    # bf16 operands: dZ is rounded to bf16 before it is multiplied, about 2e-3 of d_hidden and
    # d_weight; everything else of the step is fp32.  fp32 paths: fp32 sums over the vocabulary.
    if case["kind"] in ("step", "sft") and case["dtype"] == "bf16":
        return {"rel": 8e-3, "max": 0.1}
    return {"rel": 1.5e-5, "max": 1e-3}


# ---------------------------------------------------------------------------- oracle --
def _weights64(agg, n_i, seq, S, N):
    """Aggregation weight of each valid token: 1 / (S n_i) or 1 / N."""
    if agg == 0:
        return 1.0 / (S * n_i[seq].clamp(min=1).double())
    return torch.full(seq.shape, 1.0 / max(N, 1), dtype=torch.float64, device=DEV)


def _group64(rewards, gid, n_groups):
    """(r - mean) / (sample std + 1e-6) per group; 0 where all rewards are equal or gid < 0."""
    r, adv = rewards.double(), torch.zeros(rewards.shape, dtype=torch.float64, device=DEV)
    for k in range(n_groups):
        m = gid == k
        v = r[m]
        if v.numel() > 1 and bool((v != v[0]).any()):
            adv[m] = (v - v.mean()) / (v.std() + float(np.float32(1e-6)))
    return adv


def _ppo64(c, s, rows, seq, lp, ent, adv, T):
    """Loss, metrics, d loss / d logp and the entropy-bonus coefficients of the valid rows."""
    p = s["params"]
    n_seq = _n_seq(c)
    n_i = torch.bincount(seq, minlength=n_seq)
    ex = s["tok"].is_expert
    ex = (ex != 0) if ex is not None else torch.zeros(n_seq, dtype=torch.bool, device=DEV)
    on, exr = ~ex[seq], ex[seq]
    Non, Ne, N = int(on.sum()), int(exr.sum()), seq.numel()
    S, Son = int((n_i > 0).sum()), int(((n_i > 0) & ~ex).sum())
    w = _weights64(p.agg, n_i, seq, max(Son, 1), Non) * on
    old, ref = s["old"].double()[rows], s["ref"].double()[rows]
    A, rho = adv[seq], torch.exp(lp - old)
    pg = torch.maximum(-A * rho, -A * rho.clamp(1 - p.eps_low, 1 + p.eps_high))
    clipped = ((A > 0) & (rho > 1 + p.eps_high)) | ((A < 0) & (rho < 1 - p.eps_low))
    em1 = torch.expm1(ref - lp)
    kl = em1 - (ref - lp)
    mixed = s["tok"].is_expert is not None
    mu = p.mix_mu if mixed else 0.0
    gr = (1 - mu) * w * (torch.where(clipped, torch.zeros_like(rho), -A * rho) - p.kl_coef * em1)
    if Ne:
        gr = torch.where(exr, torch.full_like(gr, -mu / Ne), gr)
    e = (1 - mu) * p.entropy_coef * w
    pg_l, kl_l, en_l = (w * pg).sum(), (w * p.kl_coef * kl).sum(), (w * ent).sum()
    sft = (-lp * exr).sum() / max(Ne, 1)
    loss = (1 - mu) * (pg_l + kl_l - p.entropy_coef * en_l) + mu * sft
    inv, invn = 1.0 / max(Non, 1), 1.0 / max(N, 1)
    means = torch.stack([loss, pg_l, kl_l, (kl * on).sum() * inv, ent.sum() * invn,
                         (rho * on).sum() * inv, (clipped & on).double().sum() * inv])
    cnt = lambda *v: torch.tensor(v, dtype=torch.int64, device=DEV)  # noqa: E731
    return gr, e, {"means": means, "sft_loss": sft.reshape(1), "entropy_loss": en_l.reshape(1),
                   "n_valid": cnt(N, S), "n_bad_ids": cnt(0), "n_expert": cnt(Ne)}


def _full(T, rows, v):
    out = torch.zeros(T, dtype=torch.float64, device=DEV)
    out[rows] = v
    return out


def exact(case, seed):
    c, kind = case, case["kind"]
    s = prepare(case, seed)
    tok, T, V = s["tok"], s["T"], c["V"]
    for k in ("ws", "dH", "dW", "dz"):
        s.pop(k, None)
    rows = (tok.mask != 0).nonzero()[:, 0]
    seq = rows // c["pad"]
    y = tok.token_ids.long()[rows]
    N = rows.numel()
    chunk = max(1, (1 << 27) // V)

    def logits_of(rr):
        return s["H"][rr].double() @ W.t() if kind in ("step", "logprobs", "sft") else s["logits"][rr].double()

    if kind != "loss":
        if "W" in s:
            W = s["W"].double()
        lp, ent, lse = (torch.zeros(N, dtype=torch.float64, device=DEV) for _ in range(3))
        for r0 in range(0, N, chunk):
            k = slice(r0, min(N, r0 + chunk))
            z = logits_of(rows[k])
            lse[k] = torch.logsumexp(z, 1)
            lp[k] = z.gather(1, y[k][:, None])[:, 0] - lse[k]
            ent[k] = lse[k] - (torch.exp(z - lse[k][:, None]) * z).sum(1)
        out = {"logp": _full(T, rows, lp), "entropy": _full(T, rows, ent), "lse": _full(T, rows, lse)}
        if kind == "logprobs":
            return out
    e = None
    if kind == "loss":
        adv = _group64(s["rewards"], s["gid"], c["prompts"])
        gr, _, st = _ppo64(c, s, rows, seq, s["logp"].double()[rows], s["ent"].double()[rows],
                           adv, T)
        return {"adv": adv, "grad_logp": _full(T, rows, gr), "stats": st}
    if kind in ("step", "loss_logits"):
        n = _n_seq(c)
        adv = _group64(s["rewards"], torch.arange(n, device=DEV) // c["group"], c["prompts"])
        gr, e, st = _ppo64(c, s, rows, seq, lp, ent, adv, T)
        if kind == "step":
            out["adv"] = adv
    elif kind == "sft":
        n_i = torch.bincount(seq, minlength=_n_seq(c))
        S = int((n_i > 0).sum())
        w = _weights64(c["agg"], n_i, seq, max(S, 1), N)
        gr, loss = -w, (w * -lp).sum()
        zero = torch.zeros(6, dtype=torch.float64, device=DEV)
        cnt = lambda *v: torch.tensor(v, dtype=torch.int64, device=DEV)  # noqa: E731
        st = {"means": torch.cat([loss.reshape(1), zero]), "sft_loss": loss.reshape(1),
              "entropy_loss": zero[:1], "n_valid": cnt(N, S), "n_bad_ids": cnt(0),
              "n_expert": cnt(0)}
    else:
        beta, n = float(np.float32(0.1)), c["n_seq"]
        pi = torch.zeros(n, dtype=torch.float64, device=DEV).index_add_(0, seq, lp)
        rho = torch.zeros_like(pi).index_add_(0, seq, s["ref"].double()[rows])
        r = beta * (pi - rho)
        u, P = r[0::2] - r[1::2], n // 2  # every rollout has a valid token
        gs = torch.zeros_like(pi)
        gs[0::2] = -beta * torch.sigmoid(-u) / P
        gs[1::2] = beta * torch.sigmoid(-u) / P
        gr, out["seq_logp"] = gs[seq], pi
        st = {"means": torch.stack([-torch.nn.functional.logsigmoid(u).mean(), r[0::2].mean(),
                                    r[1::2].mean(), (u > 0).double().mean(), u.mean()]),
              "counts": torch.tensor([P, N, 0], dtype=torch.int64, device=DEV)}
    out["grad_logp"], out["stats"] = _full(T, rows, gr), st
    if e is not None and not float(s["params"].entropy_coef) > 0:
        e = None
    if "W" in s:
        dH = torch.zeros((T, c["d"]), dtype=torch.float64, device=DEV)
        dW = torch.zeros((V, c["d"]), dtype=torch.float64, device=DEV)
    else:
        dl = torch.zeros((T, V), dtype=torch.float64, device=DEV)
    for r0 in range(0, N, chunk):
        k = slice(r0, min(N, r0 + chunk))
        z = logits_of(rows[k])
        p = torch.exp(z - lse[k][:, None])
        dz = p * -gr[k][:, None]
        if e is not None:
            dz += e[k][:, None] * p * (z - (lse[k] - ent[k])[:, None])
        dz[torch.arange(dz.shape[0], device=DEV), y[k]] += gr[k]
        if "W" in s:
            dH[rows[k]] = dz @ W
            dW += dz.t() @ s["H"][rows[k]].double()
        else:
            dl[rows[k]] = dz
    if "W" in s:
        out["d_hidden"], out["d_weight"] = dH, dW
    else:
        out["d_logits"] = dl
    return out
