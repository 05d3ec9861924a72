"""Batches whose rollouts are mostly empty: the rollout of a row is found by a
search, not by a walk over the empty ones, and is right wherever they lie."""
import numpy as np
import pytest
import torch

import paper_2505_17826_amd as R

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _call(start, T, n_seq):
    tok = R.Tokens(torch.from_numpy(start).to(DEV), torch.ones(T, dtype=torch.uint8, device=DEV),
                   torch.zeros(T, dtype=torch.int32, device=DEV))
    adv = torch.arange(1, n_seq + 1, device=DEV).float()
    lp = torch.zeros(T, device=DEV)
    ws = torch.empty(R.workspace_bytes(R.RFT_OP_PPO_FWD, tok, 0, 5), dtype=torch.uint8, device=DEV)
    g = torch.empty(T, device=DEV)
    st = torch.zeros(R.STATS_BYTES, dtype=torch.uint8, device=DEV)
    p = R.ppo_params(0.2, 0.2, 0.0, 1)
    return lambda: R.rft_ppo_clip_loss_fwd(tok, 5, lp, lp, None, adv, p, grad_logp=g, stats=st, ws=ws)[0]


# one workgroup (starts in LDS) and several (starts in global memory)
@pytest.mark.parametrize("T,n_seq", [(8, 2000), (8, 30000), (100, 2048), (9000, 2000),
                                     (9000, 40000), (70000, 100000)])
@pytest.mark.parametrize("where", ["spread", "last", "clusters"])
def test_rollout_of_every_row(T, n_seq, where):
    print(f"[empty rollouts] T={T} n_seq={n_seq} {where}", flush=True)
    r = np.random.default_rng(T + n_seq)
    if where == "spread":
        n = np.bincount(np.sort(r.integers(0, n_seq, size=T)), minlength=n_seq)
    else:
        n = np.zeros(n_seq, np.int64)
        if where == "last":
            n[-1] = T
        else:  # runs of up to 7 empty rollouts between rollouts of a few rows
            i = 0
            while n.sum() < T and i < n_seq:
                n[i] = min(int(r.integers(1, 4)), T - n.sum())
                i += 1 + int(r.integers(0, 8))
            n[-1] += T - n.sum()
    start = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    got = _call(start, T, n_seq)().cpu().numpy()
    # ratio 1, unclipped: d loss / d logp = -advantage / T, advantage = rollout + 1
    want = -(np.repeat(np.arange(n_seq), n) + 1.0) / T
    assert np.abs(got - want).max() <= 2.0 ** -22 * np.abs(want).max()


def test_time_does_not_grow_with_empty_rollouts():
    """Eight rows among 30000 rollouts against 30000 rows of one rollout each: the
    same counts, fewer rows (a walk took 25 times as long)."""
    n_seq = 30000

    def us(fn):
        for _ in range(3):
            fn()
        ts = []
        for _ in range(15):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            fn()
            b.record()
            b.synchronize()
            ts.append(a.elapsed_time(b) * 1e3)
        return sorted(ts)[7]

    few = np.zeros(n_seq + 1, np.int32)
    few[-4000:] = np.minimum(np.arange(4000) // 500 + 1, 8)
    a, b = us(_call(few, 8, n_seq)), us(_call(np.arange(n_seq + 1, dtype=np.int32), n_seq, n_seq))
    print(f"[empty rollouts] 8 rows {a:.1f} us, {n_seq} rows {b:.1f} us", flush=True)
    assert a <= 4 * b
