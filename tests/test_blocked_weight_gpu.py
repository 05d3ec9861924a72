"""The forward GEMM from the caller's row-major weight (up to 10240 rows) and
from its tile-blocked copy on 384-row tiles (more): the same batch with and
without trailing masked rows that move it over the line gives the same bits,
through rft_token_logprobs (with the recommended and the minimum workspace) and
rft_ppo_clip_step."""
import pytest
import torch

import paper_2505_17826_amd as R

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("d,V", [(64, 300), (192, 5003), (72, 1000)])
def test_same_bits_on_both_sides(d, V):
    print(f"[blocked weight] d={d} V={V}", flush=True)
    n_seq, pad, T = 16, 640, 10240
    g = torch.Generator(device=DEV).manual_seed(d + V)
    H = torch.randn((T, d), generator=g, device=DEV).bfloat16()
    W = (torch.randn((V, d), generator=g, device=DEV) * (2 / d ** 0.5)).bfloat16()
    ids = torch.randint(0, V, (T,), generator=g, device=DEV, dtype=torch.int32)
    mask = (torch.rand(T, generator=g, device=DEV) < 0.7).to(torch.uint8)
    old = -torch.rand(T, generator=g, device=DEV) * 8
    adv = torch.randn(n_seq, generator=g, device=DEV)
    p = R.ppo_params(0.2, 0.2, 0.01, 0, entropy_coef=0.01)
    outs = []
    for extra in (0, 300):
        cat = lambda x, v: torch.cat([x, torch.full((extra, *x.shape[1:]), v, dtype=x.dtype, device=DEV)])  # noqa: E731
        start = torch.arange(n_seq + 1, dtype=torch.int32, device=DEV) * pad
        start[-1] += extra
        tok = R.Tokens(start, cat(mask, 0), cat(ids, V + 1))
        h = cat(H, float("nan"))
        o = cat(old, 0.0)
        for minimum in (False, True):
            ws = torch.empty(R.workspace_bytes(R.RFT_OP_TOKEN_LOGPROBS, tok, d, V, R.RFT_BF16,
                                               minimum=minimum), dtype=torch.uint8, device=DEV)
            outs.append([x[:T].cpu() for x in R.rft_token_logprobs(tok, h, W, ws=ws)])
        r = R.rft_ppo_clip_step(tok, h, W, o, o, adv, p)
        outs.append([x[:T].cpu() for x in r[:3]])
        full = (r[3][:T].cpu(), r[4][:T].cpu(), r[5].cpu(), r[6].cpu())
        if extra == 0:
            first = full
        else:
            for a, b in zip(first, full):
                assert torch.equal(a, b)
    for o in outs[1:]:
        for a, b in zip(outs[0], o):
            assert torch.equal(a, b)
    m = (mask != 0).cpu()
    z = H.cpu()[m].double() @ W.cpu().double().t()
    L = torch.logsumexp(z, 1)
    # fp32 sums of d exact products and of V exponentials
    assert (outs[0][2][m].double() - L).abs().max() <= (d + V / 256 + 64) * 2.0 ** -23 * (1 + z.abs().max())
