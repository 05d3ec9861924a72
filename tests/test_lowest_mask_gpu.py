"""Vocabulary entries masked by the type's lowest value give the bits of those
masked by -inf (0 probability, nothing added to the entropy, d_logits 0), also
where all the entries of a thread, a wave or a part of the row are masked:
statistics, fused call and d_logits, aligned and not, few rows and many."""
import pytest
import torch

import paper_2505_17826_amd as R

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("T,V", [(40, 5000), (40, 5003), (200, 20001), (7, 152064), (300, 152000)])
def test_lowest_value_masks_like_minus_infinity(T, V):
    print(f"[lowest mask] T={T} V={V}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(T + V)
    z = torch.randn((T, V), generator=g, device=DEV) * 3
    keep = torch.rand((T, V), generator=g, device=DEV) < 0.5
    keep[1::3] = False  # all but a window of 64 entries
    for t in range(1, T, 3):
        w = (t * 977) % (V - 64)
        keep[t, w:w + 64] = True
    keep[2::3] = True
    keep[2::3, :V // 2] = False  # the first half
    ids = keep.float().argmax(1).to(torch.int32)
    tok = R.Tokens(torch.tensor([0, T], dtype=torch.int32, device=DEV),
                   torch.ones(T, dtype=torch.uint8, device=DEV), ids)
    old = -torch.rand(T, generator=g, device=DEV) * 8
    adv = torch.ones(1, device=DEV)
    outs = []
    for low in (float("-inf"), torch.finfo(torch.float32).min):
        x = torch.where(keep, z, torch.full_like(z, low))
        st = R.rft_token_logprobs_from_logits(tok, x)[:3]
        o = list(st)
        for ent_coef in (0.0, 0.01):
            e, L, c = (torch.empty(T, device=DEV) for _ in range(3))
            p = R.ppo_params(0.2, 0.2, 0.01, entropy_coef=ent_coef)
            lp, dl, s = R.rft_ppo_clip_fused_logits(tok, x, old, old, adv, p, entropy=e, lse=L,
                                                    grad_logp=c)
            o += [lp, dl, s, e, L, c]
            kw = dict(grad_entropy=c, entropy=e) if ent_coef else {}
            o.append(R.rft_ppo_clip_loss_bwd_logits(tok, x, L, c, **kw))
            assert (dl[~keep] == 0).all() and (o[-1][~keep] == 0).all()
        outs.append(o)
    for a, b in zip(*outs):
        assert torch.equal(a, b)
    L = torch.logsumexp(torch.where(keep, z, torch.full_like(z, float("-inf"))).double(), 1)
    # V positive terms, each a few fp32 roundings of an argument below 32
    assert (outs[1][2].double() - L).abs().max() <= (V / 512 + 64) * 2.0 ** -23 * 32
