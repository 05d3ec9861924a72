"""d_hidden of an fp32 head does not depend on whether d_weight is accumulated:
few rows split the vocabulary into slices, whose partial sums lie in the
workspace, in the d_weight that is about to be overwritten or, where there is
neither, are added in turn by the same workgroups.  The bits are the same in all
three, in one chunk and in several; against float64.

Tolerance: a sum of V fp32 products in any order is off by at most
V 2^-24 sum |dz w| per element; dZ itself by the exponential's and the logit's
roundings, (d + 64) 2^-23 (1 + |z|) p."""
import pytest
import torch

import paper_2505_17826_amd as R

pytestmark = pytest.mark.gpu
DEV = "cuda"


# one row; 64 x 64 tiles with remainders; slices that end inside a K step of the
# last one; the 128 x 128 tile; a shape without slices
@pytest.mark.parametrize("T,d,V", [(1, 8, 4099), (40, 63, 5003), (5, 130, 20001), (65, 200, 3000),
                                   (2048, 1600, 6150), (300, 64, 200)])
@pytest.mark.parametrize("chunks", [1, 2])
def test_dh_bits_with_and_without_accumulation(T, d, V, chunks):
    print(f"[dh accumulate] T={T} d={d} V={V} chunks={chunks}", flush=True)
    g = torch.Generator().manual_seed(T + d + V)
    H = torch.randn((T, d), generator=g)
    W = torch.randn((V, d), generator=g) * (2 / d ** 0.5)
    ids = torch.randint(0, V, (T,), generator=g, dtype=torch.int32)
    mask = (torch.rand(T, generator=g) < 0.9).to(torch.uint8)
    mask[0] = 1
    c = torch.randn(T, generator=g) * mask
    tok = R.Tokens(torch.tensor([0, T], dtype=torch.int32, device=DEV), mask.to(DEV), ids.to(DEV))
    Hd, Wd, cd = H.to(DEV), W.to(DEV), c.to(DEV)
    _, _, lse = R.rft_token_logprobs(tok, Hd, Wd)
    rows = (T + chunks - 1) // chunks
    size = lambda f, *a: f(R.RFT_OP_PPO_BWD, tok, d, V, R.RFT_F32, *a)  # noqa: E731
    # one chunk: with and without room for the partial sums (the minimum is the
    # workspace of one chunk of 64 rows); several: the workspace of that chunk
    sizes = [size(R.workspace_bytes_rows, rows)]
    if chunks == 1:
        Tpad, Vpad = (T + 63) // 64 * 64, (V + 63) // 64 * 64
        minimum = R.workspace_bytes(R.RFT_OP_PPO_BWD, tok, d, V, R.RFT_F32, minimum=True)
        sizes.append(minimum + (Tpad - 64) * Vpad * 4)
        assert sizes[0] == R.workspace_bytes(R.RFT_OP_PPO_BWD, tok, d, V, R.RFT_F32) >= sizes[1]
        assert (sizes[0] > sizes[1]) == (V >= 256 and V // T >= 2)
        assert {size(R.chunk_rows, n) for n in sizes} == {Tpad}
    dW0 = torch.randn((V, d), generator=g).to(DEV)
    outs, dws = [], []
    for nb in sizes:
        ws = torch.empty(nb, dtype=torch.uint8, device=DEV)
        for acc in (False, True):
            dH = torch.full((T, d), float("nan"), device=DEV)
            dW = dW0.clone() if acc else torch.full((V, d), float("nan"), device=DEV)
            R.rft_ppo_clip_loss_bwd(tok, Hd, Wd, lse, cd, d_hidden=dH, d_weight=dW,
                                    accumulate_dw=acc, ws=ws)
            outs.append(dH)
            dws.append((dW, dW0.double() if acc else 0.0))
    for dH in outs[1:]:
        assert torch.equal(outs[0], dH)
    m = mask.bool().to(DEV)
    h, w, n = Hd[m].double(), Wd.double(), int(m.sum())
    z = h @ w.t()
    p = torch.exp(z - lse[m].double()[:, None])
    cm = cd[m].double()[:, None]
    dz = -cm * p
    dz[torch.arange(n, device=DEV), ids.to(DEV)[m].long()] += cd[m].double()
    eps = 2.0 ** -23
    derr = cm.abs() * p * ((d + 64) * eps * (h.abs() @ w.abs().t()) + 64 * eps * (1 + z.abs()))
    derr = derr + 4 * eps * dz.abs()
    tol = (V + 64) * eps * (dz.abs() @ w.abs()) + derr @ w.abs()
    assert ((outs[0][m].double() - dz @ w).abs() <= tol + 1e-30).all()
    assert (outs[0][~m] == 0).all()
    ref = dz.t() @ h
    tol = (n + 64) * eps * (dz.abs().t() @ h.abs()) + derr.t() @ h.abs()
    for dW, base in dws:
        r = ref + base
        assert ((dW.double() - r).abs() <= tol + 4 * eps * (r.abs() + abs(base)) + 1e-30).all()
