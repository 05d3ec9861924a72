"""The fp32 head's GEMMs at the edges of their tiles: 128 x 128 and 64 x 64
tiles, K steps of 32, remainders in every dimension, unaligned rows and bases,
and d_hidden with K split over slices, against float64 on the CPU.

Tolerance: a sum of K fp32 products in any order is off by at most
K 2^-24 sum |a b| per element (each product and each addition rounds once); the
bound below takes K + 64 in place of K for the exponentials and the loss terms."""
import pytest
import torch

import paper_2505_17826_amd as R

pytestmark = pytest.mark.gpu
DEV = "cuda"
EPS = 2.0 ** -23


def _unaligned(x, shift):
    """x on the device, its first element `shift` floats past a 16-byte boundary."""
    buf = torch.empty(x.numel() + 4, device=DEV)
    out = buf[shift:shift + x.numel()].view(x.shape)
    out.copy_(x)
    return out


# (rows, d, V): one element; tile and K-step edges +-1; the 128 x 128 tile
# (many tiles); few rows with a long K (d_hidden in slices), odd d and V
SHAPES = [(1, 1, 1), (3, 31, 63), (64, 32, 64), (65, 33, 65), (127, 64, 129), (129, 65, 127),
          (700, 130, 4100), (1500, 96, 6000), (40, 63, 5003), (5, 130, 20001)]


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("T,d,V", SHAPES)
def test_f32_head_edges(T, d, V, shift):
    print(f"[f32 head] T={T} d={d} V={V} shift={shift}", flush=True)
    g = torch.Generator().manual_seed(1000 * T + d + V)
    H = torch.randn((T, d), generator=g)
    W = torch.randn((V, d), generator=g) * (2 / d ** 0.5)
    ids = torch.randint(0, V, (T,), generator=g, dtype=torch.int32)
    mask = (torch.rand(T, generator=g) < 0.8).to(torch.uint8)
    mask[0] = 1
    c = torch.randn(T, generator=g) * mask
    m = mask.bool()
    H[~m] = float("nan")  # masked rows are never read
    tok = R.Tokens(torch.tensor([0, T], dtype=torch.int32, device=DEV), mask.to(DEV), ids.to(DEV))
    Hd, Wd = _unaligned(H, shift), _unaligned(W, shift)
    logp, ent, lse = R.rft_token_logprobs(tok, Hd, Wd)
    dW0 = torch.randn((V, d), generator=g)
    out = []
    for acc in (False, True):
        dW = dW0.to(DEV) if acc else torch.full((V, d), float("nan"), device=DEV)
        dH, dW = R.rft_ppo_clip_loss_bwd(tok, Hd, Wd, lse, c.to(DEV), d_weight=dW,
                                         accumulate_dw=acc)
        out.append((dH.cpu().double(), dW.cpu().double()))
    h, w, n = H[m].double(), W.double(), int(m.sum())
    z = h @ w.t()
    zerr = (d + 64) * EPS * (h.abs() @ w.abs().t())  # of each logit
    L = torch.logsumexp(z, 1)
    lerr = zerr.max(1).values + (V + 64) * EPS  # of the log of a sum of V positive terms
    assert ((lse.cpu()[m].double() - L).abs() <= lerr + EPS * L.abs()).all()
    zy = z[torch.arange(n), ids[m].long()]
    assert ((logp.cpu()[m].double() - (zy - L)).abs() <= 2 * lerr + 2 * EPS * (zy.abs() + L.abs())).all()
    p = torch.exp(z - lse.cpu()[m].double()[:, None])
    cm = c[m].double()[:, None]
    dz = -cm * p
    dz[torch.arange(n), ids[m].long()] += c[m].double()
    # of dZ: p (z error + a few roundings), and the rounding of c (1 - p)
    derr = cm.abs() * p * (zerr + 64 * EPS * (1 + z.abs())) + 4 * EPS * dz.abs()
    for (dH, dW), base in zip(out, (torch.zeros(V, d), dW0)):
        assert (dH[~m] == 0).all()
        tol = (V + 64) * EPS * (dz.abs() @ w.abs()) + derr @ w.abs()
        assert ((dH[m] - dz @ w).abs() <= tol + 1e-30).all()
        ref = base.double() + dz.t() @ h
        tol = (n + 64) * EPS * (dz.abs().t() @ h.abs()) + derr.t() @ h.abs() + 2 * EPS * ref.abs()
        assert ((dW - ref).abs() <= tol + EPS * base.double().abs() + 1e-30).all()
