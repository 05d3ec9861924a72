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


def test_logits_paths_of_2_23_rows():
    """One workgroup of 512 threads per row of logits: the statistics, the fused
    call and d_logits of T = 2^23 + 5 rows."""
    T, V = (1 << 23) + 5, 2
    print(f"[launch limits] logits T={T}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(2)
    logits = torch.randn((T, V), generator=g, device=DEV)
    ids = torch.randint(0, V, (T,), generator=g, device=DEV, dtype=torch.int32)
    mask = (torch.rand(T, generator=g, device=DEV) < 0.9).to(torch.uint8)
    tok = R.Tokens(torch.tensor([0, T], dtype=torch.int32, device=DEV), mask, ids)
    fill = lambda *s: torch.full(s, float("nan"), device=DEV)  # noqa: E731
    logp, ent, lse, _ = R.rft_token_logprobs_from_logits(tok, logits, logp=fill(T), entropy=fill(T),
                                                         lse=fill(T))
    m = mask.double()
    L = torch.logsumexp(logits.double(), 1)
    zy = logits.double().gather(1, ids.long()[:, None])[:, 0]
    tol = 16 * 2.0 ** -23  # a few fp32 roundings of values below 8
    assert ((lse.double() - L * m).abs() <= tol).all()
    assert ((logp.double() - (zy - L) * m).abs() <= tol).all()
    c = torch.rand(T, generator=g, device=DEV) * mask
    hot = torch.nn.functional.one_hot(ids.long(), V).double()
    want = (c.double() * m)[:, None] * (hot - torch.softmax(logits.double(), 1))
    dl = R.rft_ppo_clip_loss_bwd_logits(tok, logits, lse, c, d_logits=fill(T, V))
    assert ((dl.double() - want).abs() <= tol).all()
    adv = torch.ones(1, device=DEV)
    grad = fill(T)
    flp, fdl, st = R.rft_ppo_clip_fused_logits(tok, logits, logp, logp, adv, R.ppo_params(),
                                               logp=fill(T), grad_logp=grad, d_logits=fill(T, V))
    assert torch.equal(flp, logp)
    assert torch.equal(fdl, R.rft_ppo_clip_loss_bwd_logits(tok, logits, lse, grad))
    assert R.stats_to_dict(st)["n_valid"] == int(mask.sum())


def test_dpo_of_2_24_rollouts():
    """One workgroup of 256 threads per rollout, almost all of them empty."""
    n_seq, T = (1 << 24) + 2, 4000
    print(f"[launch limits] dpo n_seq={n_seq}", flush=True)
    start = torch.zeros(n_seq + 1, dtype=torch.int32, device=DEV)
    start[-4:] = torch.tensor([1000, 2000, 3000, 4000], dtype=torch.int32, device=DEV)
    g = torch.Generator().manual_seed(3)
    logp, ref = -torch.rand(T, generator=g).to(DEV), -torch.rand(T, generator=g).to(DEV)
    tok = R.Tokens(start, torch.ones(T, dtype=torch.uint8, device=DEV),
                   torch.zeros(T, dtype=torch.int32, device=DEV))
    _, seq, st = R.rft_dpo_loss_fwd(tok, 10, logp, ref, beta=0.125)
    pi = logp.double().view(4, 1000).sum(1)
    assert torch.equal(seq[-4:], pi.float()) or \
        (seq[-4:].double() - pi).abs().max() <= 2.0 ** -23 * pi.abs().max()
    u = 0.125 * (pi - ref.double().view(4, 1000).sum(1))
    u = u[0::2] - u[1::2]
    s = R.stats_to_dict(st, R.rft_dpo_stats)
    assert s["n_pairs"] == 2 and s["n_valid"] == T and s["n_bad_ids"] == 0
    assert math.isclose(s["loss"], float(-torch.nn.functional.logsigmoid(u).mean()), rel_tol=1e-12)


def test_advantages_of_2_24_groups():
    """One workgroup of 256 threads per group of explicit ids, one wavefront per
    group of equal size."""
    ng, n = (1 << 24) + 40, 4096
    print(f"[launch limits] groups={ng}", flush=True)
    g = torch.Generator().manual_seed(4)
    r = torch.rand(n, generator=g).to(DEV)
    gid = (ng - 1 - torch.arange(n) % 32).to(torch.int32).to(DEV)
    adv = R.rft_group_advantages_ids(r, gid, ng, mode=R.RFT_ADV_MEAN_CENTER,
                                     out=torch.full((n,), float("nan"), device=DEV))
    x = r.double().view(-1, 32)
    assert (adv.double().view(-1, 32) - (x - x.mean(0))).abs().max() <= 2.0 ** -23
    ng = (1 << 26) + 8
    r = torch.zeros(2 * ng, device=DEV)
    r[0::2] = 1
    adv = R.rft_group_advantages(r, 2, out=torch.full((2 * ng,), float("nan"), device=DEV))
    # mean 1/2, sample deviation 1/sqrt(2), eps = 1e-6
    want = 0.5 / (0.5 ** 0.5 + 1e-6)
    assert (adv[0::2] - want).abs().max() <= 2.0 ** -23
    assert (adv[1::2] + want).abs().max() <= 2.0 ** -23
