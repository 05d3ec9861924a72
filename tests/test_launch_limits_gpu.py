"""Sizes at which one work-item or workgroup per row or rollout no longer fits the
x dimension of a launch (2^32 work-items)."""
import math

import pytest
import torch

import paper_2505_17826_amd as R

pytestmark = pytest.mark.gpu
DEV = "cuda"


def test_token_logprobs_of_2_28_rows():
    """Sixteen threads per row merge the log-sum-exp partials: T = 2^28 + 40 rows,
    nearly all masked, through an fp32 head with d = 1 and V = 2."""
    T = (1 << 28) + 40
    print(f"[launch limits] T={T}", flush=True)
    rows = torch.cat([torch.arange(5), torch.arange((1 << 28) - 3, T)]).to(DEV)
    mask = torch.zeros(T, dtype=torch.uint8, device=DEV)
    mask[rows] = 1
    ids = torch.zeros(T, dtype=torch.int32, device=DEV)
    hidden = torch.zeros((T, 1), device=DEV)
    h = torch.linspace(-1, 1, rows.numel(), device=DEV)
    hidden[rows, 0] = h
    weight = torch.tensor([[1.0], [-1.0]], device=DEV)
    tok = R.Tokens(torch.tensor([0, T], dtype=torch.int32, device=DEV), mask, ids)
    logp, ent, lse = R.rft_token_logprobs(tok, hidden, weight)
    z = torch.stack([h, -h], 1).double()
    L = torch.logsumexp(z, 1)
    # two exact logits: a few fp32 roundings of values below 2
    tol = 8 * 2.0 ** -23
    assert (lse[rows].double() - L).abs().max() <= tol
    assert (logp[rows].double() - (z[:, 0] - L)).abs().max() <= tol
    H = L - (torch.softmax(z, 1) * z).sum(1)
    assert (ent[rows].double() - H).abs().max() <= tol
    for x in (logp, ent, lse):
        assert int(torch.count_nonzero(x)) <= rows.numel()
        assert int(torch.count_nonzero(x[5:(1 << 28) - 3])) == 0


@pytest.mark.parametrize("n_seq", [(1 << 24) - 1])
def test_bookkeeping_of_2_24_rollouts(n_seq):
    """One workgroup per rollout beside those of the rows' blocks: almost all
    rollouts empty, the last ones hold all the rows."""
    T, last = 100000, 1000
    print(f"[launch limits] n_seq={n_seq}", flush=True)
    start = torch.zeros(n_seq + 1, dtype=torch.int32, device=DEV)
    start[n_seq - last:] = torch.arange(last + 1, dtype=torch.int32, device=DEV) * (T // last)
    g = torch.Generator().manual_seed(1)
    mask = (torch.rand(T, generator=g) < 0.5).to(torch.uint8).to(DEV)
    logp = -torch.rand(T, generator=g).to(DEV)
    tok = R.Tokens(start, mask, torch.zeros(T, dtype=torch.int32, device=DEV))
    grad, st = R.rft_sft_loss_fwd(tok, 10, logp, agg=R.RFT_AGG_SEQ_MEAN_TOKEN_MEAN)
    n = mask.view(last, -1).double().sum(1)
    w = (mask.view(last, -1).double() / (last * n[:, None])).view(-1)
    s = R.stats_to_dict(st)
    assert s["n_valid"] == int(mask.sum()) and s["n_seq_valid"] == last
    # fp64 sums of T terms
    assert math.isclose(s["loss"], float((w * -logp.double()).sum()), rel_tol=T * 2.0 ** -53)
    assert (grad.double() + w).abs().max() <= 2.0 ** -24 * w.max()
