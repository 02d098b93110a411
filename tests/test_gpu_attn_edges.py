"""bf16 chunk attention where its tile loop can go wrong: histories and chunks
that end inside, on and just past a 64-key tile, empty histories, one to three
query tiles, whole and split items; scores whose first tile says nothing about
the others (the reference of the exponentials is taken from a segment's first
tile, and a sum or an output that it does not hold is computed again with a
running maximum); infinities and NaN.  All over a compact copy and with few
items: the split ones are cut into whole parts of one or two tiles.  Longer
parts, equal ranges of tiles and the launch that reads the cache in place are in
test_gpu_attn_redo.py."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


def _reference(Q, K, V, lens, Kq, Vq, scale):
    O, lse, bound, zmax = [], [], [], []
    for h, l in enumerate(lens):
        z = Q[h].double() @ torch.cat([K[h, :l], Kq[h]]).double().T * scale
        v = torch.cat([V[h, :l], Vq[h]]).double()
        p = torch.softmax(z, 1)
        O.append(p @ v)
        bound.append(p @ v.abs())
        lse.append(torch.logsumexp(z, 1))
        zmax.append(float(z.abs().max()))
    return torch.stack(O), torch.stack(lse), torch.stack(bound), max(zmax)


def _run(Q, K, V, lens, Kq, Vq, scale, split):
    import paper_2605_09681_amd as fkv
    n, lq, d = Q.shape
    shape = fkv.make_shape(n, d, lq, 1, 1, 1, lq, "bf16")
    ws = None
    if split:
        ws = torch.zeros(fkv.fkv_attention_workspace_size(shape), dtype=torch.uint8, device="cuda")
    O = torch.empty((n, lq, d), dtype=torch.bfloat16, device="cuda")
    lse = torch.empty((n, lq), device="cuda")
    kvl = torch.tensor(lens, dtype=torch.int32).cuda()
    for _ in range(2):      # (the counters of the first call are back at zero)
        fkv.fkv_chunk_attention(shape, Q.cuda(), K.cuda(), V.cuda(), kvl, Kq.cuda(), Vq.cuda(), scale, O, lse, ws)
    return O.cpu().double(), lse.cpu().double()


def _check(got, want, zmax):
    """P is rounded to bf16 (2^-9 each, in the output and in its normaliser), a
    part's output and the result once more each: less than 3 2^-8 of sum p |v|.
    Fp32 scores and their scaling add at most 2^-20 |z| to an exponent."""
    (O, lse), (Ow, lw, bound, _) = got, want
    tol = (3 * 2 ** -8 + zmax * 2 ** -18) * bound + 1e-30
    assert ((O - Ow).abs() <= tol).all(), float(((O - Ow).abs() / tol).max())
    assert ((lse - lw).abs() <= 2 ** -8 + zmax * 2 ** -18).all(), float((lse - lw).abs().max())


@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lq", [1, 63, 64, 65, 300, 520])
def test_tile_edges(d, lq, split):
    lens = [0, 1, 63, 64, 65, 127, 129, 640]
    g = torch.Generator().manual_seed(1000 * d + lq)
    rnd = lambda *s: torch.randn(*s, generator=g).bfloat16()
    n, slab = len(lens), 640
    Q, K, V, Kq, Vq = rnd(n, lq, d), rnd(n, slab, d), rnd(n, slab, d), rnd(n, lq, d), rnd(n, lq, d)
    for h, l in enumerate(lens):
        K[h, l:] = float("nan")         # nothing past a head's length is used
        V[h, l:] = float("nan")
    scale = 1 / math.sqrt(d)
    want = _reference(Q, K, V, lens, Kq, Vq, scale)
    _check(_run(Q, K, V, lens, Kq, Vq, scale, split), want, want[3])


@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("span", [12.0, 90.0, 400.0])
def test_scores_far_above_the_first_tile(d, span, split):
    """Each block of 64 keys has its own level of scores, `span` nats at most:
    within the reference's range, beyond 2^100, and beyond the fp32 range."""
    lens, lq = [0, 576, 600, 1024], 130
    g = torch.Generator().manual_seed(int(d + span))
    n, slab = len(lens), 1024
    rnd = lambda *s: torch.randn(*s, generator=g)
    scale = 1 / math.sqrt(d)
    u = torch.ones(d) / math.sqrt(d)
    Q = (rnd(n, lq, d) * 0.5 + 4 * u).bfloat16()          # component 4 along u
    level = torch.rand(n, (slab + lq + 63) // 64, generator=g).repeat_interleave(64, 1)[:, :slab + lq] * span
    keys = (rnd(n, slab + lq, d) * 0.5 + (level / (4 * scale))[..., None] * u).bfloat16()
    K, Kq = keys[:, :slab].contiguous(), keys[:, slab:].contiguous()
    V, Vq = rnd(n, slab, d).bfloat16(), rnd(n, lq, d).bfloat16()
    want = _reference(Q, K, V, lens, Kq, Vq, scale)
    _check(_run(Q, K, V, lens, Kq, Vq, scale, split), want, want[3])


@pytest.mark.parametrize("split", [False, True])
def test_infinities_and_nan_stay_in_their_place(split):
    d, lq, slab, lens = 128, 70, 256, [200, 256, 256]
    g = torch.Generator().manual_seed(5)
    rnd = lambda *s: torch.randn(*s, generator=g).bfloat16()
    Q, K, V, Kq, Vq = rnd(3, lq, d), rnd(3, slab, d), rnd(3, slab, d), rnd(3, lq, d), rnd(3, lq, d)
    V[0, 130, 7] = float("inf")
    V[1, 100, 3] = float("nan")
    Q[2, 5, 0] = float("nan")
    scale = 1 / math.sqrt(d)
    O, lse = _run(Q, K, V, lens, Kq, Vq, scale, split)
    Ow, lw, bound, zmax = _reference(Q, K, V, lens, Kq, Vq, scale)
    bad = torch.zeros_like(O, dtype=torch.bool)
    bad[0, :, 7] = bad[1, :, 3] = bad[2, 5] = True
    assert (O[0, :, 7] == float("inf")).all()
    assert O[1, :, 3].isnan().all() and O[2, 5].isnan().all()
    tol = 3 * 2 ** -8 * bound + 1e-5
    assert ((O - Ow).abs() <= tol)[~bad].all()
    rows = torch.ones(3, lq, dtype=torch.bool)
    rows[2, 5] = False
    assert ((lse - lw).abs() <= 2 ** -8)[rows].all()
