"""d_hidden of few rows through a bf16 head, whose K (the vocabulary) is split
into slices: one row, rows around a 256-row tile, hidden sizes around a tile and
small vocabularies (one slice), and many rows, of which only the last, partial
round of tiles is cut; against float64; the same bits whichever tile
RFT_GEMM_STORE_TILE fixes.

Tolerance: dZ is rounded to bf16 (a relative 2^-9 per element; its fp32 value is
off by the exponential's error, far below that), then a sum of V exact products
in fp32, off by at most V 2^-24 sum |dz w| in any order."""
import pytest
import torch

import paper_2505_17826_amd as R

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("T,d,V", [(1, 8, 4096), (255, 264, 20000), (257, 248, 33000),
                                   (40, 1032, 9000), (700, 72, 40001), (1030, 512, 2049),
                                   (130, 64, 65), (18100, 4096, 2000), (17800, 4000, 1500)])
def test_dh_slices(T, d, V, monkeypatch):
    print(f"[slices] T={T} d={d} V={V}", flush=True)
    g = torch.Generator().manual_seed(T + d + V)
    H = torch.randn((T, d), generator=g).bfloat16()
    W = (torch.randn((V, d), generator=g) * (2 / d ** 0.5)).bfloat16()
    ids = torch.randint(0, V, (T,), generator=g, dtype=torch.int32)
    mask = (torch.rand(T, generator=g) < 0.7).to(torch.uint8)
    mask[0] = 1
    m = mask.bool()
    c = torch.randn(T, generator=g) * mask
    H[~m] = float("nan")
    tok = R.Tokens(torch.tensor([0, T], dtype=torch.int32, device=DEV), mask.to(DEV), ids.to(DEV))
    Hd, Wd = H.to(DEV), W.to(DEV)
    _, _, lse = R.rft_token_logprobs(tok, Hd, Wd)
    outs = []
    for tile in ("256", "384", None):
        if tile is None:
            monkeypatch.delenv("RFT_GEMM_STORE_TILE", raising=False)
        else:
            monkeypatch.setenv("RFT_GEMM_STORE_TILE", tile)
        dH = torch.full((T, d), float("nan"), device=DEV)
        R.rft_ppo_clip_loss_bwd(tok, Hd, Wd, lse, c.to(DEV), d_hidden=dH)
        outs.append(dH)
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    m, lse, ids = m.to(DEV), lse.double(), ids.to(DEV)
    c = c.to(DEV)
    h, w, n = Hd[m].double(), Wd.double(), int(m.sum())
    z = h @ w.t()
    cm = c[m].double()[:, None]
    p = torch.exp(z - lse[m][:, None])
    dz = -cm * p
    dz[torch.arange(n, device=DEV), ids[m].long()] += c[m].double()
    # d roundings of each logit and the exponential's, relative to p
    perr = (d + 64) * 2.0 ** -23 * (h.abs() @ w.abs().t()) + 64 * 2.0 ** -23 * (1 + z.abs())
    tol = (2.0 ** -8 + (V + 64) * 2.0 ** -23) * (dz.abs() @ w.abs()) + (cm.abs() * p * perr) @ w.abs()
    got = outs[0]
    assert (got[~m] == 0).all()
    assert ((got[m].double() - dz @ w).abs() <= tol + 1e-30).all()
