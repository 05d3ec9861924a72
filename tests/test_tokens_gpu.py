"""Token bookkeeping at the edges of its paths: one workgroup (up to 8192 rows
and 2048 rollouts), one block of 2048 rows more or less, the counts added by
each block or scanned (past 2^21 rows), loss sums of one block, of many and of
more than the last block adds; masks at odd addresses, empty rollouts, expert
flags.  Counts are exact; the loss is the fp64 mean over valid tokens of values
that are exact in fp32, so only its rounding order differs (1e-12 relative)."""
import numpy as np
import pytest
import torch

import paper_2505_17826_amd as R

pytestmark = pytest.mark.gpu
DEV = "cuda"

CASES = [(1, 1), (7, 3), (256, 8), (257, 300), (2048, 2049), (8191, 5), (8192, 2048), (8193, 7),
         (10240, 2049), (300001, 400), (700000, 33), ((1 << 21) + 5, 4099)]


@pytest.mark.parametrize("shift", [0, 3])
@pytest.mark.parametrize("T,n_seq", CASES)
def test_counts_and_loss_sums(T, n_seq, shift):
    print(f"[tokens] T={T} n_seq={n_seq} shift={shift}", flush=True)
    r = np.random.default_rng(T + n_seq)
    cuts = np.sort(r.integers(0, T + 1, size=n_seq - 1))  # some rollouts are empty
    start = np.concatenate([[0], cuts, [T]]).astype(np.int32)
    mask = (r.random(T) < 0.6).astype(np.uint8) * r.integers(1, 256, size=T).astype(np.uint8)
    expert = (r.random(n_seq) < 0.3).astype(np.uint8)
    ids = r.integers(0, 50, size=T).astype(np.int32)
    bad = r.random(T) < 0.01
    ids[bad] = 50
    lp = -(r.integers(1, 64, size=T) / 8.0).astype(np.float32)
    buf = torch.empty(T + 8, dtype=torch.uint8, device=DEV)
    m = buf[shift:shift + T]
    m.copy_(torch.from_numpy(mask))
    t = lambda x: torch.from_numpy(x).to(DEV)  # noqa: E731
    tok = R.Tokens(t(start), m, t(ids), t(expert))
    grad, st = R.rft_ppo_clip_loss_fwd(tok, 50, t(lp), t(lp), None, torch.ones(n_seq, device=DEV),
                                       R.ppo_params(0.2, 0.2, 0.0, 1, mix_mu=0.5))
    s = R.stats_to_dict(st)
    sg, sst = R.rft_sft_loss_fwd(tok, 50, t(lp), agg=0)
    ss = R.stats_to_dict(sst)
    v = mask != 0
    seq = np.searchsorted(start[1:], np.arange(T), side="right")
    n_i = np.bincount(seq[v], minlength=n_seq)
    ex = expert[seq] != 0
    N, S, Ne = int(v.sum()), int((n_i > 0).sum()), int((v & ex).sum())
    for d in (s, ss):
        assert (d["n_valid"], d["n_seq_valid"], d["n_bad_ids"]) == (N, S, int((v & bad).sum()))
    assert s["n_expert"] == Ne
    use = v & ~bad
    Ng = N - Ne
    g = np.zeros(T)
    if Ng:
        g[use & ~ex] = -0.5 / Ng
    if Ne:
        g[use & ex] = -0.5 / Ne
    assert np.array_equal(grad.cpu().numpy(), g.astype(np.float32))
    sft = -lp[use & ex].astype(np.float64).sum() / max(Ne, 1)
    assert abs(s["sft_loss"] - sft) <= 1e-12 * abs(sft)
    w = np.zeros(T)
    w[use] = 1.0 / (S * n_i[seq[use]].astype(np.float64))
    assert np.array_equal(sg.cpu().numpy(), (-w).astype(np.float32))
    want = (w * -lp.astype(np.float64)).sum()
    assert abs(ss["loss"] - want) <= 1e-12 * max(want, 1e-300)


@pytest.mark.parametrize("mode", [R.RFT_ADV_GRPO, R.RFT_ADV_MEAN_CENTER, R.RFT_ADV_LEAVE_ONE_OUT])
@pytest.mark.parametrize("n,n_groups", [(1, 1), (3, 2), (256, 300), (257, 31), (511, 3), (512, 64),
                                        (513, 64), (1023, 1), (1024, 64), (1025, 64)])
def test_advantages_of_few_rollouts(n, n_groups, mode):
    """One launch up to 512 rollouts, the bucketed path past them: fp64 sums
    rounded once to fp32 (2^-24 of the result; 1e-12 for the sums' order)."""
    r = np.random.default_rng(7 * n + mode)
    rew = r.random(n).astype(np.float32)
    rew[r.random(n) < 0.3] = 1.0
    gid = r.integers(-1, n_groups + 1, size=n).astype(np.int32)
    got = R.rft_group_advantages_ids(torch.from_numpy(rew).to(DEV), torch.from_numpy(gid).to(DEV),
                                     n_groups, mode).cpu().numpy()
    want = np.zeros(n)
    for g in range(n_groups):
        k = gid == g
        v = rew[k].astype(np.float64)
        if v.size < 2 or (mode == R.RFT_ADV_GRPO and v.min() == v.max()):
            continue
        if mode == R.RFT_ADV_GRPO:
            want[k] = (v - v.mean()) / (v.std(ddof=1) + float(np.float32(1e-6)))
        elif mode == R.RFT_ADV_MEAN_CENTER:
            want[k] = v - v.mean()
        else:
            want[k] = v - (v.sum() - v) / (v.size - 1)
    assert (np.abs(got - want) <= 2.0 ** -23 * np.abs(want) + 1e-12).all()


def test_advantages_take_the_faster_path():
    """1000 rollouts by buckets, like 1500 (by one launch they took 1.6 times as long)."""

    def us(n):
        rew = torch.rand(n, device=DEV)
        gid = torch.randint(0, n // 8, (n,), device=DEV, dtype=torch.int32)
        ws = torch.empty(R.lib().rft_group_advantages_ids_workspace_bytes(n, n // 8),
                         dtype=torch.uint8, device=DEV)
        out = torch.empty_like(rew)
        ts = []
        for i in range(25):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(8):
                R.rft_group_advantages_ids(rew, gid, n // 8, out=out, ws=ws)
            b.record()
            b.synchronize()
            ts.append(a.elapsed_time(b) * 125)
        return sorted(ts)[8]

    us(1000)
    a, b = us(1000), us(1500)
    print(f"[advantages] 1000: {a:.1f} us, 1500: {b:.1f} us", flush=True)
    assert a <= 1.35 * b
