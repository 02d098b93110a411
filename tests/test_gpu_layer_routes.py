"""The routes of a compacting layer step: one stream or two, timed or not."""
import numpy as np
import pytest
import torch

import workloads as W
from gpu_harness import dev_inputs, make_layer

pytestmark = pytest.mark.gpu

_SLOT = np.array([3, 0, 8, 1, 5, 2, 7], np.int32)


def _small(dtype="bf16"):
    S, D = W.STATIC, W.DYNAMIC
    heads = (W.HeadBudget(S, 1, 2), W.HeadBudget(D, 1, 0, 2, W.SCOPE_FRAME), W.HeadBudget(D, 0, 1, 3, W.SCOPE_GLOBAL),
             W.HeadBudget(S, 0, 3))
    cfg = W.LayerConfig("small", len(heads), 64, 100, 7, 9, 2, 25, dtype, heads, 0.85)
    return cfg, W.make_layer_inputs(cfg, seed=40, frame_slot=_SLOT)


@pytest.mark.parametrize("two", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_events_time_the_step_that_runs(dtype, two):
    """A step with events launches what the step without them does: the same
    output bits, the same compressed copy, every named launch timed."""
    cfg, x = _small(dtype)
    d = dev_inputs(x)
    got = []
    for timed in (False, True):
        layer = make_layer(cfg, step_mode="compact")
        layer.two_streams = two
        names = layer.attention_launches()
        assert names == (("static_attention", "dynamic_attention") if two else ("attention",))
        events = {n: tuple(torch.cuda.Event(enable_timing=True) for _ in range(2)) for n in names} if timed else None
        O = torch.empty_like(d["Q"])
        lse = torch.empty((cfg.n_heads, cfg.lq), dtype=torch.float32, device="cuda")
        layer.step(d["K_hist"], d["V_hist"], x.frame_slot, d["Q"], d["K_cur"], d["V_cur"], O, lse, events=events)
        torch.cuda.synchronize()
        for a, b in (events or {}).values():
            assert a.elapsed_time(b) > 0
        got.append((O, lse, layer.scores, layer.kept_seg, layer.kv_len, layer.Kc, layer.Vc))
    for a, b in zip(*got):
        assert torch.equal(a, b)


def test_the_caller_chooses_the_route():
    """Small layers take one stream by themselves; overlap="always", an explicit
    in_place=True or a slab without room for the static heads takes two."""
    cfg, x = _small()
    heads = (W.HeadBudget(W.STATIC, 1, 6),) + cfg.heads[1:]          # keeps all 700 tokens, the dynamic heads 400
    route = lambda **kw: make_layer(cfg, heads, step_mode="compact", **kw).two_streams
    assert not route() and not route(overlap=False) and not route(in_place=False) and not route(slab=700)
    assert route(overlap="always") and route(in_place=True) and route(slab=400)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_compress_on_two_streams(dtype):
    """compress() with overlap="always": the bytes of the one-stream call."""
    cfg, x = _small(dtype)
    d = dev_inputs(x)
    got = []
    for overlap in (True, "always"):
        layer = make_layer(cfg, step_mode="compact", overlap=overlap)
        layer.compress(d["K_hist"], d["V_hist"], x.frame_slot, d["K_cur"])
        torch.cuda.synchronize()
        got.append((layer.scores, layer.kept_seg, layer.kv_len, layer.Kc, layer.Vc))
    for a, b in zip(*got):
        assert torch.equal(a, b)
