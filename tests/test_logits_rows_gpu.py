"""The loss-only kernels over the lengths and alignments of a row: the edges of
the on-chip variants (chunks of 2048 logits: 6, 17, 31 and 73-75 of them), a
handful of rows cut into parts, rows
whose start and length are no multiple of 16 bytes, d_logits aligned unlike the
logits, very short rows; the fused, statistics-only and d_logits-only calls give
the same bits, and float64's values.

Tolerance: fp32 exponentials and sums of V positive terms in an order of about
V / 512 steps: (V / 512 + 64) 2^-23 relative on sums, the same absolute on lse."""
import pytest
import torch

import paper_2505_17826_amd as R

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _at(x, shift):
    buf = torch.empty(x.numel() + 4, device=DEV)
    out = buf[shift:shift + x.numel()].view(x.shape)
    out.copy_(x)
    return out


@pytest.mark.parametrize("ent", [0.0, 0.02])
@pytest.mark.parametrize("T,V,shift,dshift", [
    (24, 1, 0, 0), (24, 2, 3, 1), (24, 3, 1, 0), (24, 5, 2, 2), (24, 2047, 0, 0),
    (24, 6 * 2048, 0, 1), (24, 6 * 2048 + 1, 1, 1), (24, 17 * 2048 + 3, 0, 0),
    (200, 17 * 2048 + 4, 2, 0), (200, 31 * 2048, 0, 0), (160, 31 * 2048 + 7, 3, 3),
    (160, 75 * 2048 - 2, 0, 0), (160, 73 * 2048 + 9, 1, 2),
    # rows cut into 8, 4 and 2 parts
    (12, 37449, 0, 0), (12, 37450, 1, 0), (32, 75 * 2048 - 2, 0, 0), (33, 73 * 2048 + 9, 1, 2),
    (64, 31 * 2048 + 7, 3, 3), (65, 65536, 0, 1), (128, 65537, 2, 2), (129, 65536, 0, 0)])
def test_row_lengths_and_alignments(T, V, shift, dshift, ent):
    print(f"[row] T={T} V={V} shift={shift} dshift={dshift} ent={ent}", flush=True)
    g = torch.Generator().manual_seed(V + shift)
    z0 = torch.randn((T, V), generator=g) * 2
    if V > 4:
        z0[3, ::3] = float("-inf")  # masked vocabulary entries
    ids = torch.randint(0, V, (T,), generator=g, dtype=torch.int32)
    ids[3] = 1 if V > 4 else ids[3]
    ids[5] = V  # out of range
    mask = torch.ones(T, dtype=torch.uint8)
    mask[[0, 7, 8]] = 0
    z0[0] = float("nan")  # masked rows are never read
    m = mask.bool()
    z = _at(z0, shift)
    start = torch.tensor([0, 8, T // 2 + 3, T], dtype=torch.int32, device=DEV)
    tok = R.Tokens(start, mask.to(DEV), ids.to(DEV))
    t = lambda x: x.to(DEV)  # noqa: E731
    zm = z0[m].double()
    L = torch.logsumexp(zm, 1)
    y = ids[m].long()
    ok = (y >= 0) & (y < V)
    lp = torch.where(ok, zm.gather(1, y.clamp(max=V - 1)[:, None])[:, 0] - L, torch.nan)
    old, ref = torch.zeros(T), torch.zeros(T)
    old[m] = (torch.nan_to_num(lp) + 0.05).float()
    ref[m] = (torch.nan_to_num(lp) - 0.1).float()
    adv = torch.tensor([1.0, -0.5, 0.25])
    p = R.ppo_params(0.2, 0.2, 0.01, 0, entropy_coef=ent)
    e1 = lambda: torch.empty(T, device=DEV)  # noqa: E731
    flp, fent, flse, fgr = e1(), e1(), e1(), e1()
    dl = _at(torch.full((T, V), float("nan")), dshift)
    R.rft_ppo_clip_fused_logits(tok, z, t(old), t(ref), t(adv), p, logp=flp, entropy=fent, lse=flse,
                                grad_logp=fgr, d_logits=dl)
    ulp, uent, ulse, _ = R.rft_token_logprobs_from_logits(tok, z)
    eg = torch.empty(T, device=DEV)
    ugr, _ = R.rft_ppo_clip_loss_fwd(tok, V, ulp, t(old), t(ref), t(adv), p, entropy=uent,
                                     grad_entropy=eg)
    udl = R.rft_ppo_clip_loss_bwd_logits(tok, z, ulse, ugr, grad_entropy=eg if ent else None,
                                         entropy=uent if ent else None)
    for a, b in ((flp, ulp), (fent, uent), (flse, ulse), (fgr, ugr), (dl, udl)):
        assert torch.equal(torch.nan_to_num(a, nan=7.0), torch.nan_to_num(b, nan=7.0))
    eps = (V / 512 + 64) * 2.0 ** -23
    P = torch.exp(zm - L[:, None])
    H = -(P * torch.where(P > 0, zm - L[:, None], torch.zeros_like(zm))).sum(1)
    assert ((flse.cpu()[m].double() - L).abs() <= eps * (1 + L.abs())).all()
    assert ((fent.cpu()[m].double() - H).abs() <= eps * (1 + zm.nan_to_num(neginf=0).abs().max(1).values) * 4).all()
    assert torch.isnan(flp.cpu()[m][~ok]).all()
    c, e = fgr.cpu()[m].double()[:, None], eg.cpu()[m].double()[:, None]
    onehot = torch.zeros_like(zm)
    onehot[torch.arange(len(y)), y.clamp(max=V - 1)] = ok.double()
    zf = torch.where(P > 0, zm, torch.zeros_like(zm))
    want = c * (onehot - P) + e * P * (zf - (L - H)[:, None]) * (P > 0)
    tol = (c.abs() * (P + onehot) + e * P * (1 + zf.abs() + L[:, None].abs())) * 8 * eps * (1 + L.abs().max())
    got = dl.cpu()
    assert (got[~m] == 0).all()
    assert ((got[m].double() - want).abs() <= tol + 1e-30).all()
