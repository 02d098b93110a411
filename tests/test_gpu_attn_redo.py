"""bf16 chunk attention where a segment is computed again with a running
maximum, under every schedule (one workgroup per item, items cut into whole
parts, equal ranges of key tiles over items of unequal length) and through
both entry points: over a compact copy, and read in place from the cache with
pieces that are no multiple of a 64-key tile."""
import math

import numpy as np
import pytest
import torch

from test_gpu_attn_edges import _check

pytestmark = pytest.mark.gpu

F, H, C = 90, 20, 6                  # 540 query rows: three query tiles, the last of 28 rows
LQ, QT = C * F, 3


def _kept_frames(schedule):
    """History frames of each head."""
    if schedule == "ranges":         # 9, 37, 10, 36, 12 and 16 tiles in turn
        return [[0, 20, 1, 19, 2, 5][h % 6] for h in range(48)]
    if schedule == "parts":          # two parts of 18 and 19 tiles
        return [20] * 42
    return [20, 0, 7, 13]            # one workgroup per item, or parts of one or two tiles


def _tiles(kept):
    return [-(-(k * F + LQ) // 64) for k in kept]


def _segments(kept):
    """The balanced schedule's segments, as lists of (item, t0, t1, tiles of the
    item) per workgroup, and whether items are cut into whole parts."""
    G = max(8, torch.cuda.get_device_properties(0).multi_processor_count // 8 * 8)
    items = [t for t in _tiles(kept) for _ in range(QT)]
    total = sum(items)
    parts = G // len(items)
    if parts >= 2 and -(-max(items) // parts) <= total // min(G, total) + 4:
        cut = [(i, T * j // min(parts, T), T * (j + 1) // min(parts, T), T)
               for i, T in enumerate(items) for j in range(min(parts, T))]
        return [[s] for s in cut], True
    G = min(G, total)
    bases = np.concatenate([[0], np.cumsum(items)])
    out = []
    for r in range(G):
        lo, hi = r * total // G, (r + 1) * total // G
        segs = []
        while lo < hi:
            i = int(np.searchsorted(bases, lo, "right")) - 1
            t1 = min(hi, int(bases[i + 1]))
            segs.append((i, lo - int(bases[i]), t1 - int(bases[i]), items[i]))
            lo = t1
        out.append(segs)
    return out, False


def _check_schedule(schedule, kept):
    """The schedule reaches what the case is for."""
    segs, whole = _segments(kept)
    longest = max(t1 - t0 for s in segs for _, t0, t1, _ in s)
    if schedule == "ranges":
        assert not whole
        # a workgroup that computes a whole item and goes on, whose last V tile lies in
        # a buffer that the next segment's first two tiles are stored into
        assert any((T - 1) % 4 in (0, 1) and t1 - t0 == T for s in segs for _, t0, t1, T in s[:-1])
        assert any(t1 - t0 < T and t1 - t0 > 2 for s in segs for _, t0, t1, T in s)
    elif schedule == "parts":
        assert whole and longest > 10
    elif schedule == "short-parts":
        assert whole and longest <= 2


class _Inputs:
    """Histories kept in the cache (head h static, or dynamic with its kept
    segments written out) and the same histories gathered."""

    def __init__(self, schedule, d, seed, keys, Q):
        import paper_2605_09681_amd as fkv
        import workloads as W
        self.kept = kept = _kept_frames(schedule)
        _check_schedule(schedule, kept)
        self.fkv, self.d, self.n = fkv, d, len(kept)
        self.split = schedule != "items"
        rng = np.random.default_rng(seed)
        g = torch.Generator().manual_seed(seed)
        self.slots = rng.permutation(H).astype(np.int32)
        self.lens = [k * F for k in kept]
        self.Q = Q(g, self.n)
        self.K, self.Kq = keys(g, self.n, kept)          # [n][H*F][d]: kept rows first, then others; [n][LQ][d]
        self.V = torch.randn(self.n, H * F, d, generator=g).bfloat16()
        self.Vq = torch.randn(self.n, LQ, d, generator=g).bfloat16()
        self.shape = fkv.make_shape(self.n, d, F, H, H, C, F, "bf16")
        budgets, self.kept_seg = [], torch.full((self.n, H), -1, dtype=torch.int32)
        self.K_hist, self.V_hist = torch.empty(self.n, H, F, d).bfloat16(), torch.empty(self.n, H, F, d).bfloat16()
        for h, k in enumerate(kept):
            if h % 2 == 0:
                budgets.append(W.HeadBudget(W.STATIC, min(k, 1), max(k - 1, 0)))
                frames = list(range(min(k, 1))) + list(range(H - max(k - 1, 0), H))
            else:
                budgets.append(W.HeadBudget(W.DYNAMIC, 0, 0, k, W.SCOPE_GLOBAL))
                frames = sorted(rng.permutation(H)[:k].tolist())
                self.kept_seg[h, :k] = torch.tensor(frames, dtype=torch.int32)
            order = frames + [t for t in range(H) if t not in frames]
            for y, t in enumerate(order):
                self.K_hist[h, self.slots[t]] = self.K[h, y * F:(y + 1) * F]
                self.V_hist[h, self.slots[t]] = self.V[h, y * F:(y + 1) * F]
        self.heads = fkv.make_heads(budgets)

    def run(self):
        """O and lse of both entry points (each called twice: the counters of
        the first call are back at zero); the two agree bit for bit."""
        fkv, shape, dev = self.fkv, self.shape, lambda t: t.cuda()
        ws = (torch.zeros(fkv.fkv_attention_workspace_size(shape), dtype=torch.uint8, device="cuda")
              if self.split else None)
        Kc, Vc = self.K.clone(), self.V.clone()
        for h, l in enumerate(self.lens):
            Kc[h, l:] = float("nan")
            Vc[h, l:] = float("nan")
        kvl = torch.tensor(self.lens, dtype=torch.int32).cuda()
        Q, Kq, Vq = dev(self.Q), dev(self.Kq), dev(self.Vq)
        scale, outs = 1 / math.sqrt(self.d), []
        Kc, Vc, Kh, Vh, seg = dev(Kc), dev(Vc), dev(self.K_hist), dev(self.V_hist), dev(self.kept_seg)
        for call in ("compact", "paged"):
            O, lse = torch.empty_like(Q), torch.empty((self.n, LQ), device="cuda")
            for _ in range(2):
                if call == "compact":
                    fkv.fkv_chunk_attention(shape, Q, Kc, Vc, kvl, Kq, Vq, scale, O, lse, ws)
                else:
                    fkv.fkv_chunk_attention_paged(shape, self.heads, Kh, Vh, self.slots, seg, kvl, Q, Kq, Vq, scale,
                                                  O, lse, ws)
            outs.append((O.cpu(), lse.cpu()))
        (Oc, lc), (Op, lp) = outs
        assert torch.equal(Oc.view(torch.int16), Op.view(torch.int16))
        assert torch.equal(lc.view(torch.int32), lp.view(torch.int32))
        return Oc.double(), lc.double()

    def reference(self):
        """In fp64 on the device; |z| of the scores that can weigh anything."""
        scale, O, lse, bound, zmax = 1 / math.sqrt(self.d), [], [], [], 0.0
        for h, l in enumerate(self.lens):
            k = torch.cat([self.K[h, :l], self.Kq[h]]).cuda().double()
            v = torch.cat([self.V[h, :l], self.Vq[h]]).cuda().double()
            z = self.Q[h].cuda().double() @ k.T.contiguous() * scale
            p = torch.softmax(z, 1)
            O.append((p @ v).cpu())
            bound.append((p @ v.abs()).cpu())
            lse.append(torch.logsumexp(z, 1).cpu())
            zmax = max(zmax, float(z[z > -1e6].abs().max()))
        return torch.stack(O), torch.stack(lse), torch.stack(bound), zmax


SCHEDULES = ["items", "short-parts", "parts", "ranges"]


@pytest.mark.parametrize("schedule", SCHEDULES)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("span", [40.0, 90.0, 400.0])
def test_levels_above_the_reference(d, span, schedule):
    """Every frame and every 64 keys of the chunk have a level of scores of their
    own, `span` nats apart at most, the chunk's last 64 keys the lowest: sums of up
    to 2^57 (their exponent goes to the part's maximum), above 2^100, and beyond
    the fp32 range (both computed again)."""
    print(f"[gpu case] attention-levels d={d} span={span} schedule={schedule}", flush=True)
    scale, u = 1 / math.sqrt(d), torch.ones(d) / math.sqrt(d)

    def queries(g, n):
        return (torch.randn(n, LQ, d, generator=g) * 0.5 + 4 * u).bfloat16()     # component 4 along u

    def keys(g, n, kept):
        hist = torch.rand(n, H, generator=g).repeat_interleave(F, 1)
        chunk = torch.rand(n, -(-LQ // 64), generator=g).repeat_interleave(64, 1)[:, :LQ]
        chunk[:, -64:] = 0
        level = torch.cat([hist, chunk], 1) * span
        k = (torch.randn(n, H * F + LQ, d, generator=g) * 0.5 + (level / (4 * scale))[..., None] * u).bfloat16()
        return k[:, :H * F].contiguous(), k[:, H * F:].contiguous()

    x = _Inputs(schedule, d, int(d + span), keys, queries)
    want = x.reference()
    _check(x.run(), want, want[3])


@pytest.mark.parametrize("schedule", SCHEDULES)
@pytest.mark.parametrize("base", [0.0, 150.0, -150.0])
@pytest.mark.parametrize("mask", [float("-inf"), -3.3895313892515355e38, -1e30])
def test_keys_with_the_lowest_scores(mask, base, schedule):
    """Keys that weigh nothing -- -inf, a bf16 lowest value whose products overflow
    to it, or a large negative value -- where they fill whole tiles and parts: the
    ragged last tile, the chunk's first 150 rows, every third frame.  The other
    scores lie around `base` nats, so a reference of 0 would not hold them."""
    print(f"[gpu case] attention-lowest mask={mask} base={base} schedule={schedule}", flush=True)
    d = 64 if schedule == "ranges" and base else 128

    def queries(g, n):
        return (torch.rand(n, LQ, d, generator=g) + 0.5).bfloat16()              # every product has the mask's sign

    def keys(g, n, kept):
        k = torch.randn(n, H * F + LQ, d, generator=g) * 0.3 + base / math.sqrt(d)
        k[:, H * F:H * F + 150] = mask
        k[:, -63:] = mask
        k[:, :H * F].view(n, H, F, d)[:, ::3] = mask
        k = k.bfloat16()
        return k[:, :H * F].contiguous(), k[:, H * F:].contiguous()

    x = _Inputs(schedule, d, int(200 + base), keys, queries)
    want = x.reference()
    assert want[0].isfinite().all()
    _check(x.run(), want, want[3])


@pytest.mark.parametrize("schedule", SCHEDULES)
def test_infinities_and_nan_in_recomputed_segments(schedule):
    """An infinite or NaN value, and a NaN query, reach what they weigh in and
    nothing else, whichever segments are computed again for them."""
    print(f"[gpu case] attention-infinities schedule={schedule}", flush=True)
    d = 64

    def queries(g, n):
        q = torch.randn(n, LQ, d, generator=g).bfloat16()
        q[2, 5, 0] = float("nan")
        return q

    def keys(g, n, kept):
        return torch.randn(n, H * F, d, generator=g).bfloat16(), torch.randn(n, LQ, d, generator=g).bfloat16()

    x = _Inputs(schedule, d, 11, keys, queries)
    x.Vq[0, 130, 7], x.Vq[1, 100, 3] = float("inf"), float("nan")
    O, lse = x.run()
    bad = torch.zeros_like(O, dtype=torch.bool)
    bad[0, :, 7] = bad[1, :, 3] = bad[2, 5] = True
    assert (O[0, :, 7] == float("inf")).all() and O[1, :, 3].isnan().all() and O[2, 5].isnan().all()
    assert lse[2, 5].isnan()
    x.Q, x.Vq = x.Q.nan_to_num(), x.Vq.nan_to_num(posinf=0.0)
    Ow, lw, bound, zmax = x.reference()
    O, lse = torch.where(bad, Ow, O), torch.where(bad[:, :, 0], lw, lse)
    _check((O, lse), (Ow, lw, bound, zmax), zmax)
