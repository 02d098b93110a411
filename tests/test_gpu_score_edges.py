"""Segment scores where the reduction's route changes: units of up to 16 column
groups (128 tokens of 128 bf16 channels, 64 of fp32) have one partial per arrival
group and are added by the head's last workgroup, longer ones go through group
sums.  Both sides of the edge, one and several units, unit counts that shift a
unit's groups, and the history statistics with cached scores."""
import pytest
import torch

pytestmark = pytest.mark.gpu

_DT = {"bf16": torch.bfloat16, "f32": torch.float32}


@pytest.mark.parametrize("dtype,d,L,units", [("bf16", 128, 1, 3), ("bf16", 128, 9, 31), ("bf16", 128, 128, 3),
                                             ("bf16", 128, 129, 3), ("bf16", 64, 256, 2), ("bf16", 64, 257, 1),
                                             ("f32", 128, 64, 5), ("f32", 128, 65, 5)])
def test_scores_on_both_sides_of_the_direct_sum(dtype, d, L, units):
    """Every sum is fp64 over exact products, the cosine is rounded once to fp32:
    within one fp32 step (2^-23, |score| <= 1) of fp64; cached scores the same bits."""
    import paper_2605_09681_amd as fkv
    import workloads as W
    H, C, n, F = 5, 1, 3, L * units
    g = torch.Generator().manual_seed(7 * L + units)
    K = torch.randn(n, H, F, d, generator=g).to(_DT[dtype])
    Kq = (K[:, -1] * 0.7 + torch.randn(n, F, d, generator=g) * 0.5).to(_DT[dtype])
    slots = [3, 0, 4, 1, 2]
    cache = torch.empty_like(K)
    cache[:, slots] = K
    x = torch.cat([K, Kq[:, None]], 1).double().reshape(n, H + 1, units, L * d)
    sq, dot = (x * x).sum(-1), (x[:, :-1] * x[:, 1:]).sum(-1)
    want = (dot / (sq[:, :-1] * sq[:, 1:]).sqrt()).reshape(n, -1)
    shape = fkv.make_shape(n, d, F, H, H, C, L, dtype)
    heads = fkv.make_heads([W.HeadBudget(W.DYNAMIC, 0, 0, 1, W.SCOPE_GLOBAL)] * n)
    scores = torch.zeros((n, H * units), device="cuda")
    dev = cache.cuda(), Kq.cuda()
    ws = fkv.fkv_score_segments(shape, heads, dev[0], slots, dev[1], scores)
    first = scores.cpu()
    assert (first.double() - want).abs().max() <= 2 ** -23
    fkv.fkv_score_segments(shape, heads, dev[0], slots, dev[1], scores, ws)
    assert torch.equal(scores.cpu(), first)
    stats = torch.zeros(fkv.fkv_score_stats_size(shape, heads) // 8, dtype=torch.float64, device="cuda")
    fkv.fkv_score_history(shape, heads, dev[0], slots, stats, ws)
    scores.zero_()
    fkv.fkv_score_segments_cached(shape, heads, dev[0], slots, dev[1], stats, scores, ws)
    assert torch.equal(scores.cpu(), first)
