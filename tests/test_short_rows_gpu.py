"""d_logits of short rows (up to 1024 logits: one wavefront per row, four rows per
workgroup) and of the first longer ones: rows that are no multiple of four, odd
lengths and alignments, masked rows, ids out of range and in each part of a row;
against float64, with and without the entropy term.

Tolerance: p is an exponential of a rounded argument below 32 in size
(2^-23 * 32 relative), then a few fp32 roundings."""
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


@pytest.mark.parametrize("ent", [False, True])
@pytest.mark.parametrize("T,V,shift,dshift", [
    (1, 1, 0, 0), (5, 2, 1, 0), (7, 3, 2, 3), (9, 4, 0, 0), (6, 7, 3, 1), (41, 255, 0, 1),
    (40, 256, 0, 0), (43, 257, 1, 1), (39, 260, 0, 0), (30, 511, 2, 0), (29, 1020, 0, 0),
    (31, 1023, 3, 2), (33, 1024, 0, 0), (35, 1025, 0, 0), (37, 2049, 1, 3), (300, 4100, 0, 0)])
def test_short_rows(T, V, shift, dshift, ent):
    print(f"[short rows] T={T} V={V} shift={shift} dshift={dshift} ent={ent}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(T + V)
    z = _at(torch.randn((T, V), generator=g, device=DEV) * 2, shift)
    ids = torch.randint(0, V, (T,), generator=g, device=DEV, dtype=torch.int32)
    ids[0], ids[T // 2], ids[T - 1] = 0, V - 1, V
    mask = (torch.rand(T, generator=g, device=DEV) < 0.8).to(torch.uint8)
    mask[0] = 1
    tok = R.Tokens(torch.tensor([0, T], dtype=torch.int32, device=DEV), mask, ids)
    zd = z.double()
    L = torch.logsumexp(zd, 1)
    P = torch.exp(zd - L[:, None])
    H = (P * (L[:, None] - zd)).sum(1)
    c = torch.randn(T, generator=g, device=DEV)
    e = torch.rand(T, generator=g, device=DEV) if ent else torch.zeros(T, device=DEV)
    lse, entropy = L.float(), H.float()
    dl = _at(torch.full((T, V), float("nan")), dshift)
    kw = dict(grad_entropy=e, entropy=entropy) if ent else {}
    R.rft_ppo_clip_loss_bwd_logits(tok, z, lse, c, d_logits=dl, **kw)
    P = torch.exp(zd - lse.double()[:, None])
    hot = torch.nn.functional.one_hot(ids.clamp(max=V - 1).long(), V).double() * (ids < V)[:, None]
    mu = (lse - entropy).double()[:, None]
    want = c.double()[:, None] * (hot - P) + e.double()[:, None] * P * (zd - mu)
    want = want * mask.double()[:, None]
    tol = 40 * 2.0 ** -23 * (c.double().abs()[:, None] * (hot + P)
                             + e.double()[:, None] * P * (1 + zd.abs() + mu.abs()))
    assert ((dl.double() - want).abs() <= tol + 1e-30).all()
    assert (dl[mask == 0] == 0).all()


def test_time_of_short_rows():
    """The same number of logits in rows of 25 and of 500: short rows cost their
    count of rows, but not a workgroup of 512 threads each (20 times as long)."""

    def us(T, V):
        z = torch.randn((T, V), device=DEV)
        dl = torch.empty_like(z)
        x = torch.rand(T, device=DEV)
        tok = R.Tokens(torch.tensor([0, T], dtype=torch.int32, device=DEV),
                       torch.ones(T, dtype=torch.uint8, device=DEV),
                       torch.zeros(T, dtype=torch.int32, device=DEV))
        for _ in range(3):
            R.rft_ppo_clip_loss_bwd_logits(tok, z, x, x, d_logits=dl)
        ts = []
        for _ in range(15):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(4):
                R.rft_ppo_clip_loss_bwd_logits(tok, z, x, x, d_logits=dl)
            b.record()
            b.synchronize()
            ts.append(a.elapsed_time(b) * 250)
        return sorted(ts)[7]

    a, b = us(96000, 25), us(4800, 500)
    print(f"[short rows] rows of 25 {a:.1f} us, of 500 {b:.1f} us", flush=True)
    assert a <= 5 * b
