"""Attention mass at the sizes where its bins and tiles can go wrong: bins that
share a 64-key tile (up to 32 keys), bins shorter than, equal to and just past
one, histories that are not a
whole number of bins, more bins than keys, several query tiles, accumulation."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("F,C", [(1, 5), (1, 300), (2, 40), (3, 7), (21, 13), (31, 9), (32, 9), (33, 8), (63, 1), (64, 5), (65, 4), (130, 3)])
def test_mass_edges(d, F, C):
    """Every head's mass against fp64 softmax column sums.  The probabilities
    are fp32 exponentials of fp32 score sums (|z| < 32, so each is within
    about d 2^-24 |z| + 2^-22 of its value, far below 1e-4), added in fp32."""
    import paper_2605_09681_amd as fkv
    H = 6
    slab = H * F
    lens = [0, 1, slab // 2 + 1, slab - 1, slab, slab + 9]
    n, lq, extra = len(lens), C * F, 3
    g = torch.Generator().manual_seed(100 * d + F)
    rnd = lambda *s: torch.randn(*s, generator=g).bfloat16()
    Q, K, Kq = rnd(n, lq, d), rnd(n, slab, d), rnd(n, lq, d)
    scale = 1 / math.sqrt(d)
    n_bins = -(-(slab + lq) // F) + extra
    want, lse = torch.zeros(n, n_bins, dtype=torch.float64), torch.empty(n, lq)
    for h, l in enumerate(lens):
        z = Q[h].double() @ torch.cat([K[h, :l], Kq[h]]).double().T * scale
        lse[h] = torch.logsumexp(z, 1).float()
        p = torch.softmax(z, 1).sum(0)
        K[h, l:] = float("nan")
        for b in range(-(-p.numel() // F)):
            want[h, b] = p[b * F:(b + 1) * F].sum()
    shape = fkv.make_shape(n, d, F, H, H, C, F, "bf16")
    kvl = torch.tensor(lens, dtype=torch.int32).cuda()
    mass = torch.full((n, n_bins), 7.0, device="cuda")
    args = (shape, Q.cuda(), K.cuda(), kvl, Kq.cuda(), lse.cuda(), scale, mass)
    ws = fkv.fkv_attention_mass(*args)
    first = mass.cpu()
    err = (first.double() - want).abs()
    assert (err <= 1e-4 * want + 1e-5 * lq).all(), float((err / (1e-4 * want + 1e-5 * lq)).max())
    assert (first[want == 0] == 0).all()
    fkv.fkv_attention_mass(*args, accumulate=True, workspace=ws)
    assert torch.equal(mass.cpu(), first * 2)      # the same bits again
