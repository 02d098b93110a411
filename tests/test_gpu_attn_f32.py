"""fp32 chunk attention (fp32 matrix cores) at the sizes where its tiling can
go wrong: 32-query row blocks, 32-key tiles dealt to eight waves, the tile
that straddles history and chunk, and waves that get no tile."""
import math

import pytest
import torch

from gpu_harness import F32_MAX_ABS, F32_REL_L2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("F", [1, 31, 33, 70])
def test_attention_f32_edges(d, F):
    """Every row and the log normaliser against fp64, with history lengths
    around the tile edges (0 to past the slab: clamped), rows past kv_len
    poisoned with NaN, queries scaled for sharp rows."""
    import paper_2605_09681_amd as fkv
    lens = [0, 1, 31, 32, 33, 64, 223, 224, 225, 257, 300, 999, -3]
    slab = 300
    n = len(lens)
    g = torch.Generator().manual_seed(1000 * d + F)
    rnd = lambda *s: torch.randn(*s, generator=g)
    Q, K, V = 3 * rnd(n, F, d), rnd(n, slab, d), rnd(n, slab, d)
    Kq, Vq = rnd(n, F, d), rnd(n, F, d)
    for h, l in enumerate(lens):
        K[h, max(l, 0):] = float("nan")
        V[h, max(l, 0):] = float("nan")
    scale = 1 / math.sqrt(d)
    shape = fkv.make_shape(n, d, F, 4, 4, 1, F, "f32")
    dev = lambda t: t.cuda()
    O, lse = torch.empty(n, F, d, device="cuda"), torch.empty(n, F, device="cuda")
    fkv.fkv_chunk_attention(shape, dev(Q), dev(K), dev(V), dev(torch.tensor(lens, dtype=torch.int32)), dev(Kq),
                            dev(Vq), scale, O, lse)
    for h, l in enumerate(lens):
        m = min(max(l, 0), slab)
        k, v = torch.cat([K[h, :m], Kq[h]]).double(), torch.cat([V[h, :m], Vq[h]]).double()
        z = Q[h].double() @ k.T * scale
        ref, rl = torch.softmax(z, 1) @ v, torch.logsumexp(z, 1)
        err = O[h].cpu().double() - ref
        assert err.abs().max() <= F32_MAX_ABS and err.norm() <= F32_REL_L2 * ref.norm(), (l, err.abs().max())
        assert (lse[h].cpu().double() - rl).abs().max() <= 1e-5, l


def test_attention_f32_infinite_scores():
    """Keys whose scores are -inf weigh nothing, also when they fill a tile or
    a wave's whole share; a NaN key poisons exactly the rows that see it."""
    import paper_2605_09681_amd as fkv
    n, d, F, slab = 2, 64, 40, 96
    g = torch.Generator().manual_seed(5)
    Q = torch.rand(n, F, d, generator=g) + 0.5
    K, V = torch.randn(n, slab, d, generator=g), torch.randn(n, slab, d, generator=g)
    Kq, Vq = torch.randn(n, F, d, generator=g), torch.randn(n, F, d, generator=g)
    K[0, :70] = -float("inf")          # q . k = -inf for positive q
    K[1, 50, 3] = float("nan")
    shape = fkv.make_shape(n, d, F, 4, 4, 1, F, "f32")
    kvl = torch.full((n,), slab, dtype=torch.int32).cuda()
    O = torch.empty(n, F, d, device="cuda")
    fkv.fkv_chunk_attention(shape, Q.cuda(), K.cuda(), V.cuda(), kvl, Kq.cuda(), Vq.cuda(), 0.125, O)
    k, v = torch.cat([K[0, 70:], Kq[0]]).double(), torch.cat([V[0, 70:], Vq[0]]).double()
    ref = torch.softmax(Q[0].double() @ k.T * 0.125, 1) @ v
    assert (O[0].cpu().double() - ref).norm() <= F32_REL_L2 * ref.norm()
    assert O[1].isnan().all()
