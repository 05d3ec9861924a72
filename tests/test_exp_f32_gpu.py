"""The exponentials of the fp32 head.  With one row, hidden size 1, hidden = 1,
a given log-sum-exp of 0 and d loss / d logp = -1, d_weight[v] is exp(weight[v])
itself (one product by 1, and sums of zeros), so the backward shows each
exponential's own rounding.

Bound: a library exponential is within 1 ulp; 2 ulps are allowed, each ulp
2^-23 of the value or, below the normal range, 2^-149.  Taking exp2 of the rounded product x log2(e)
instead is off by up to 15 half-ulps at x = -15 and loses the subnormal results."""
import pytest
import torch

import paper_2505_17826_amd as R

pytestmark = pytest.mark.gpu
DEV = "cuda"


# V: the 64 x 64 tile with a remainder, and enough columns for every range of x
@pytest.mark.parametrize("lo,hi,V", [(-1.0, 0.0, 4097), (-10.0, -1.0, 20000), (-20.0, -10.0, 20000),
                                     (-87.0, -20.0, 20000), (-103.0, -87.4, 2000)])
def test_exponential_is_as_exact_as_the_librarys(lo, hi, V):
    print(f"[exp f32] [{lo}, {hi}] V={V}", flush=True)
    g = torch.Generator().manual_seed(V)
    x = lo + (hi - lo) * torch.rand((V, 1), generator=g)
    x[0] = 0.0  # the sampled token's entry, left out below
    tok = R.Tokens(torch.tensor([0, 1], dtype=torch.int32, device=DEV),
                   torch.ones(1, dtype=torch.uint8, device=DEV),
                   torch.zeros(1, dtype=torch.int32, device=DEV))
    one = torch.ones((1, 1), device=DEV)
    _, dW = R.rft_ppo_clip_loss_bwd(tok, one, x.to(DEV), torch.zeros(1, device=DEV),
                                    -torch.ones(1, device=DEV))
    got = dW.cpu().double()[1:, 0]
    want = torch.exp(x.double())[1:, 0]
    ulp = torch.clamp(want * 2.0 ** -23, min=2.0 ** -149)
    err = (got - want) / ulp
    assert err.abs().max() <= 2.0, float(err.abs().max())
    # no common bias, which would add up over a vocabulary: a rounding of at most
    # half an ulp either way averages out to well below a tenth of one
    assert abs(float(err.mean())) <= 0.1 or hi < -87, float(err.mean())
