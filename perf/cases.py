"""Timing cases of the Forcing-KV hot path: what a streaming video-diffusion
program has this package do, over the range of sizes it is used at.

A case is a dict of plain values; ``kind`` says which public call it makes:

* ``step``      one layer, one AR step (``CompressedLayer.step``): score and
                select the dynamic heads' segments, attend every head;
* ``fp8``       the same with the FP8 attention (``CompressedLayer.step_fp8``);
* ``chunk``     one chunk of a rollout (``RolloutStack``): every layer's AR
                steps, then the write of the finished chunk into the cache;
* ``score``     scoring and selection alone (``CompressedLayer.score_select``);
* ``compress``  scoring, selection and the gathered copy (``.compress``);
* ``observe``   one observation of the offline head profiling
                (``HeadProfiler.observe``).

Sizes: F tokens per frame, H history frames in cap slots, C chunk frames,
segments of L tokens; ``n_static`` of ``heads`` heads are static (sink frame +
``recent`` frames), the others dynamic (sink frame + the fraction ``keep`` of
the segments, per frame when L < F).  Wan-1.3B shapes: 12 heads of 128, 1560
tokens per frame at 480P, 8160 at 1080P, 21-frame window, 3-frame chunks.
"""
import math

import numpy as np
import torch

import workloads as W
from paper_2605_09681_amd.layer import CompressedLayer, HeadProfiler, RolloutStack

_DT = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(name, kind, **kw):
    c = dict(kind=kind, dtype="bf16", heads=12, d=128, F=1560, H=21, cap=21, C=3, L=1560, n_static=6,
             sink=1, recent=6, keep=0.5, lse=False)
    if kind == "chunk":
        c.update(layers=2, steps=4, scoring="own", index=1)
    if name:
        c["name"] = name
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: the package's tiny fp32 configuration, launch-bound (unit tests, CPU-size models)
        _case("tiny-f32", "step", dtype="f32", heads=2, d=64, F=64, H=4, cap=4, C=1, L=64, n_static=1, recent=1,
              sink=0, keep=0.5, lse=True),
        # a small model with head_dim 64 and ragged sizes: tiles and pieces that end inside a frame
        _case("small-d64", "step", heads=16, d=64, F=333, H=13, cap=16, C=2, L=111, n_static=8, recent=3, lse=True),
        # a rollout's second chunk: 3 history frames, little to compress
        _case("chunk-early-480p", "chunk", H=3, index=1, recent=1),
        # a long rollout's chunk at the full window: history statistics once, 4 AR steps, 2 layers
        _case("chunk-480p", "chunk", index=9, scoring="incremental"),
        # the headline unit: one 480P layer step, one frame per segment
        _case("step-480p", "step"),
        # the same with quarter-frame segments selected per frame, a quarter kept (a point of the keep sweep)
        _case("step-480p-L390", "step", L=390, keep=0.25),
        # the headline unit at 1080P: the largest
        _case("step-1080p", "step", F=8160, L=8160),
        # the FP8 step at 480P: selection, packing from the cache, FP8 attention
        _case("fp8-480p", "fp8"),
        # scoring and selection alone, as a program overlaps it with other work
        _case("score-480p", "score"),
        # segments too short to be attended in place: the gathered copy
        _case("compress-480p-L52", "compress", L=52),
        # offline head profiling: one 480P observation over the whole history
        _case("observe-480p", "observe"),
        # an fp32 layer at a quarter of the 480P tokens (parity runs against a bf16 model)
        _case("step-f32", "step", dtype="f32", F=390, L=390),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        kind = rng.choice(["step"] * 5 + ["chunk"] * 3 + ["fp8"] * 2 + ["score", "compress", "observe"])
        f32 = kind in ("step", "score", "compress") and rng.random() < 0.2
        seg = rng.choice(["frame", "frame", "sub", "multi"])
        if seg == "sub":
            n = rng.randint(2, 12)
            L = log_int(24, 800)
            F = n * L
        else:
            F = log_int(64, 4096)
            L = F if seg == "frame" else F * rng.randint(2, 4)
        heads = rng.randint(2, 16)
        C = rng.randint(1, 4)
        H = rng.randint(2, 24)
        c = _case(None, kind, dtype="f32" if f32 else "bf16", heads=heads, d=rng.choice([64, 128, 128]), F=F, H=H,
                  cap=H + rng.randint(0, 3), C=C, L=L, n_static=rng.randint(1, heads - 1), recent=rng.randint(1, 6),
                  keep=round(rng.uniform(0.15, 0.8), 2), lse=kind in ("step", "fp8") and rng.random() < 0.3)
        if kind == "chunk":
            index = rng.randint(1, 9)
            window = max(C + 1, H)
            c.update(layers=rng.randint(1, 2), steps=rng.randint(1, 4), index=index, cap=window,
                     scoring=rng.choice(["own", "incremental", "pooled"]), H=min(index * C, window))
        if kind == "observe":
            c.update(L=F)
        if F > 8160 or -(-c["H"] * F // L) > 4096:
            continue
        w = work(c)
        if w["flops"] <= (4e10 if f32 else 2e12) and w["bytes"] <= 1.5e9:
            return c


# ------------------------------------------------------------------ budgets
def _segments(c):
    return -(-c["H"] * c["F"] // c["L"])


def _heads(c):
    H, F, L = c["H"], c["F"], c["L"]
    if L < F:
        k, scope = int(F // L * c["keep"] + 1e-9), W.SCOPE_FRAME
    else:
        sink_segs = min(-(-c["sink"] // (L // F)), _segments(c))
        k, scope = int((_segments(c) - sink_segs) * c["keep"] + 1e-9), W.SCOPE_GLOBAL
    st = W.HeadBudget(W.STATIC, c["sink"] or 1, c["recent"])
    dy = W.HeadBudget(W.DYNAMIC, c["sink"], 0, k, scope)
    return [st] * c["n_static"] + [dy] * (c["heads"] - c["n_static"])


def _static_frames(b, H):
    return sorted(set(range(min(b.sink_frames, H))) | set(range(max(H - b.recent_frames, 0), H)))


def _tokens(c, b):
    """Retained history tokens of a head (the largest number, where a short last segment makes it depend on scores)."""
    H, F, L = c["H"], c["F"], c["L"]
    if b.type == W.STATIC:
        return len(_static_frames(b, H)) * F
    n, kept = _segments(c), 0
    if b.scope == W.SCOPE_FRAME:
        per = F // L
        kept = min(b.sink_frames, H) * per + max(H - b.sink_frames, 0) * min(b.keep_k, per)
    else:
        sink = sum(1 for g in range(n) if g * L // F < b.sink_frames)
        kept = sink + min(b.keep_k, n - sink)
    return min(kept * L, H * F)


# --------------------------------------------------------------------- work
def work(case):
    c = case
    es = 2 if c["dtype"] == "bf16" else 4
    row = c["d"] * es
    lq, H, F, n = c["C"] * c["F"], c["H"], c["F"], c["heads"]
    heads = _heads(c)
    kept = [_tokens(c, b) for b in heads]
    n_dyn = sum(b.type == W.DYNAMIC for b in heads)
    if c["kind"] == "score":
        return {"bytes": n_dyn * ((H + 1) * F * row + _segments(c) * 8), "flops": n_dyn * (H + 1) * F * c["d"] * 4}
    if c["kind"] == "compress":
        dyn = sum(k for k, b in zip(kept, heads) if b.type == W.DYNAMIC)
        read = n_dyn * (H + 1) * F + dyn + 2 * (sum(kept) - dyn)    # K of all, V of the kept; static K and V
        return {"bytes": row * (read + 2 * sum(kept)), "flops": n_dyn * (H + 1) * F * c["d"] * 4}
    if c["kind"] == "observe":
        return {"bytes": n * row * (2 * H * F + 4 * lq) + n * lq * 4, "flops": 4 * n * lq * (H * F + lq) * c["d"]}
    chunk = 4 * n * lq * row + (n * lq * 4 if c["lse"] else 0)       # Q, K_cur, V_cur, O
    flops = 4 * lq * c["d"] * sum(k + lq for k in kept)
    dyn = sum(k for k, b in zip(kept, heads) if b.type == W.DYNAMIC)
    if c["kind"] != "chunk":
        return {"bytes": row * (n_dyn * H * F + dyn + 2 * (sum(kept) - dyn)) + chunk, "flops": flops}
    steps = c["steps"] * (2 * sum(kept) * row + chunk)
    scored = {"own": c["layers"] * c["steps"] * (n_dyn * H * F - dyn), "incremental": c["layers"] * n_dyn * H * F,
              "pooled": c["steps"] * n * H * F}[c["scoring"]] * row
    return {"bytes": c["layers"] * (steps + 4 * n * lq * row) + scored, "flops": c["layers"] * c["steps"] * flops}


def tolerance(case):
    if case["kind"] in ("score", "compress"):
        return "exact"
    if case["kind"] == "fp8":
        return {"rel": 0.03, "max": 0.9}     # probabilities in 3 mantissa bits
    if case["dtype"] == "f32":
        return {"rel": 6e-6, "max": 2e-4}
    return {"rel": 1e-2, "max": 0.2}


# ------------------------------------------------------------------- inputs
def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(g, shape, dt):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).to(dt)


def _keys(g, n, frames, F, d, dt):
    """Keys of consecutive frames, similar from one to the next by a degree that differs per head and token."""
    rho = 0.8 + 0.18 * torch.rand((n, F, 1), generator=g, device="cuda")
    out = torch.empty((n, frames, F, d), dtype=dt, device="cuda")
    k = None
    for t in range(frames):
        eps = torch.randn((n, F, d), generator=g, device="cuda")
        k = eps if k is None else rho * k + (1 - rho * rho).sqrt() * eps
        out[:, t] = k.to(dt)
    return out


def _slots(c, seed):
    if c["kind"] == "chunk":
        return W.ring_frame_slots(c["index"], c["C"], c["cap"])
    if c["H"] == c["cap"]:            # a rotated ring with its first slot pinned
        r = 1 + seed % max(c["cap"] - 1, 1)
        return np.array([0] + list(range(r, c["cap"])) + list(range(1, r)), np.int32)[:c["H"]]
    return np.random.default_rng(seed).permutation(c["cap"])[:c["H"]].astype(np.int32)


def _layer_inputs(c, seed, extra_chunks=1):
    """K_hist, V_hist in their slots, and per AR step (Q, K_cur, V_cur)."""
    g, dt = _generator(seed), _DT[c["dtype"]]
    n, d, F, H, C = c["heads"], c["d"], c["F"], c["H"], c["C"]
    slots = _slots(c, seed)
    at = torch.from_numpy(np.asarray(slots, np.int64)).cuda()
    chain = _keys(g, n, H + C, F, d, dt)
    K = _normal(g, (n, c["cap"], F, d), dt)
    V = _normal(g, (n, c["cap"], F, d), dt)
    K[:, at] = chain[:, :H]
    steps = []
    for s in range(extra_chunks):
        kq = chain[:, H:].reshape(n, C * F, d).contiguous()
        if s:                         # the chunk is denoised further at each step
            kq = (0.95 * kq.float() + 0.3 * _normal(g, kq.shape, torch.float32)).to(dt)
        steps.append((_normal(g, kq.shape, dt), kq, _normal(g, kq.shape, dt)))
    return K, V, slots, steps


def prepare(case, seed):
    c = case
    n, d, F, H, C = c["heads"], c["d"], c["F"], c["H"], c["C"]
    if c["kind"] == "chunk":
        stack = RolloutStack(c["layers"], n, d, F, c["cap"], C, c["L"], c["dtype"])
        steps = []
        for layer in range(c["layers"]):
            K, V, slots, st = _layer_inputs(c, seed * 8 + layer, c["steps"])
            stack.K_hist[layer].copy_(K)
            stack.V_hist[layer].copy_(V)
            steps.append([(*x, torch.empty_like(x[0])) for x in st])
        return dict(case=c, stack=stack, slots=slots, steps=steps, budgets=_heads(c),
                    dst=W.chunk_write_slots(c["index"], C, c["cap"]))
    K, V, slots, steps = _layer_inputs(c, seed)
    Q, Kq, Vq = steps[0]
    s = dict(case=c, K=K, V=V, slots=slots, Q=Q, Kq=Kq, Vq=Vq)
    if c["kind"] == "observe":
        s["profiler"] = HeadProfiler(n, d, F, H, c["cap"], C)
        return s
    s["layer"] = CompressedLayer(n, d, F, H, c["cap"], C, c["L"], c["dtype"], _heads(c))
    s["O"] = torch.empty_like(Q)
    s["lse"] = torch.empty((n, C * F), dtype=torch.float32, device="cuda") if c["lse"] else None
    if c["kind"] == "fp8":
        s["layer"].fp8_buffers()
    return s


# ---------------------------------------------------------------------- run
def run(state):
    s, c = state, state["case"]
    if c["kind"] == "chunk":
        stack, slots = s["stack"], s["slots"]
        incremental = c["scoring"] == "incremental"
        if incremental:
            for layer in range(c["layers"]):
                stack.history(layer, s["budgets"], slots)
        for k in range(c["steps"]):
            row = None
            for layer in range(c["layers"]):
                Q, Kq, Vq, O = s["steps"][layer][k]
                if c["scoring"] == "pooled" and layer == 0:
                    row = stack.score_pooled(0, slots, Kq)
                stack.run_layer(layer, s["budgets"], slots, Q, Kq, Vq, O, pooled=row, incremental=incremental)
        for layer in range(c["layers"]):
            _, Kq, Vq, _ = s["steps"][layer][-1]
            stack.append(layer, Kq, Vq, s["dst"])
        return {"O": [[st[3] for st in layer] for layer in s["steps"]], "K": list(stack.K_hist), "V": list(stack.V_hist)}
    if c["kind"] == "observe":
        p = s["profiler"]
        p.observed = 0                # the first observation of a profile
        p.observe(s["Q"], s["K"], s["V"], s["slots"], s["Kq"], s["Vq"])
        return {"mass": p.mass, "O": p.O, "lse": p.lse}
    layer = s["layer"]
    if c["kind"] == "score":
        layer.score_select(s["K"], s["slots"], s["Kq"])
        return {"scores": layer.scores, "kept_seg": layer.kept_seg, "kv_len": layer.kv_len}
    if c["kind"] == "compress":
        layer.compress(s["K"], s["V"], s["slots"], s["Kq"])
        return {"Kc": layer.Kc, "Vc": layer.Vc, "scores": layer.scores, "kept_seg": layer.kept_seg,
                "kv_len": layer.kv_len}
    step = layer.step_fp8 if c["kind"] == "fp8" else layer.step
    step(s["K"], s["V"], s["slots"], s["Q"], s["Kq"], s["Vq"], s["O"], s["lse"])
    out = {"O": s["O"], "scores": layer.scores, "kept_seg": layer.kept_seg}
    if s["lse"] is not None:
        out["lse"] = s["lse"]
    return out


# -------------------------------------------------------------------- exact
def _scores64(c, K, slots, Kq, pooled=False):
    """[heads (1 when pooled)][segments] cosines of adjacent frames, rounded to fp32."""
    H, F, L, d = c["H"], c["F"], c["L"], c["d"]
    U = min(L, F)
    dots, sqs = [], []
    for h in range(K.shape[0]):
        x = torch.cat([K[h][torch.from_numpy(np.asarray(slots, np.int64)).cuda()], Kq[h, :F].reshape(1, F, d)]).double()
        x = x.reshape(H + 1, F // U, U * d)
        sqs.append((x * x).sum(-1))
        dots.append((x[:-1] * x[1:]).sum(-1))
    dot, sq = torch.stack(dots), torch.stack(sqs)
    if pooled:
        dot, sq = dot.sum(0, keepdim=True), sq.sum(0, keepdim=True)
    na, nb = sq[:, :-1], sq[:, 1:]
    if L > F:
        m = L // F
        pad = -H % m

        def group(v):
            v = torch.nn.functional.pad(v[..., 0], (0, pad))
            return v.reshape(v.shape[0], -1, m).sum(-1)
        dot, na, nb = group(dot), group(na), group(nb)
    p = na * nb
    return torch.where(p == 0, torch.zeros_like(p), dot / p.sqrt()).reshape(dot.shape[0], -1).float()


def _kept(c, b, row):
    """Ascending kept segments of a dynamic head from its score row."""
    H, F, L, n = c["H"], c["F"], c["L"], _segments(c)
    s = row.tolist()
    frames = [(g * L // F, (min(g * L + L, H * F) - 1) // F) for g in range(n)]
    forced = [f < b.sink_frames or e >= H - b.recent_frames for f, e in frames]
    keep = {g for g in range(n) if forced[g]}
    groups = {}
    for g in range(n):
        if not forced[g]:
            groups.setdefault(frames[g][0] if b.scope == W.SCOPE_FRAME else 0, []).append(g)
    for members in groups.values():
        keep |= set(sorted(members, key=lambda g: (s[g], g))[:b.keep_k])
    return sorted(keep)


def _gather(c, b, X, slots, kept):
    """A head's retained rows of X [cap][F][d] in logical order."""
    at = torch.from_numpy(np.asarray(slots, np.int64)).cuda()
    x = X[at].reshape(-1, c["d"])
    if b.type == W.STATIC:
        runs = [(t * c["F"], (t + 1) * c["F"]) for t in _static_frames(b, c["H"])]
    else:
        runs = [(g * c["L"], min((g + 1) * c["L"], c["H"] * c["F"])) for g in kept]
    return torch.cat([x[a:e] for a, e in runs]) if runs else x[:0]


def _attend64(q, k, v, scale, F=0):
    """Output and log normaliser of one head in fp64, and the mass of each block of F keys."""
    k, v = k.double(), v.double()
    O, lse, mass = [], [], 0.0
    rows = max(64, min(q.shape[0], 150_000_000 // max(k.shape[0], 1)))
    for i in range(0, q.shape[0], rows):
        z = (q[i:i + rows].double() @ k.T).mul_(scale)
        l = torch.logsumexp(z, 1)
        p = z.sub_(l[:, None]).exp_()
        O.append(p @ v)
        lse.append(l)
        if F:
            mass = mass + p.sum(0).reshape(-1, F).sum(1)
    return torch.cat(O), torch.cat(lse), mass


def exact(case, seed):
    c = case
    heads, scale = _heads(c), 1 / math.sqrt(c["d"])
    n, n_seg = c["heads"], _segments(c)

    def layer(K, V, slots, Q, Kq, Vq, row=None, attend=True):
        scores = torch.zeros((n, n_seg), dtype=torch.float32, device="cuda")
        kept_seg = torch.full((n, n_seg), -1, dtype=torch.int32)
        own = None if row is not None else _scores64(c, K[c["n_static"]:], slots, Kq[c["n_static"]:])
        O, lse, rows = [], [], []
        for h, b in enumerate(heads):
            kept = []
            if b.type == W.DYNAMIC:
                r = row if row is not None else own[h - c["n_static"]]
                scores[h] = r
                kept = _kept(c, b, r)
                kept_seg[h, :len(kept)] = torch.tensor(kept, dtype=torch.int32)
            if attend is not None:
                rows.append((_gather(c, b, K[h], slots, kept), _gather(c, b, V[h], slots, kept)))
            if attend:
                o, l, _ = _attend64(Q[h], torch.cat([rows[-1][0], Kq[h]]), torch.cat([rows[-1][1], Vq[h]]), scale)
                O.append(o)
                lse.append(l)
        return scores, kept_seg, rows, O, lse

    if c["kind"] == "chunk":
        outs, Ks, Vs, pooled = [], [], [], []
        for i in range(c["layers"]):
            K, V, slots, steps = _layer_inputs(c, seed * 8 + i, c["steps"])
            if i == 0 and c["scoring"] == "pooled":
                pooled = [_scores64(c, K, slots, kq, pooled=True)[0] for _, kq, _ in steps]
            outs.append([torch.stack(layer(K, V, slots, *st, row=pooled[k] if pooled else None)[3])
                         for k, st in enumerate(steps)])
            dst = torch.from_numpy(np.asarray(W.chunk_write_slots(c["index"], c["C"], c["cap"]), np.int64)).cuda()
            K[:, dst] = steps[-1][1].reshape(n, c["C"], c["F"], c["d"])
            V[:, dst] = steps[-1][2].reshape(n, c["C"], c["F"], c["d"])
            Ks.append(K)
            Vs.append(V)
        return {"O": outs, "K": Ks, "V": Vs}
    K, V, slots, steps = _layer_inputs(c, seed)
    Q, Kq, Vq = steps[0]
    if c["kind"] == "observe":
        at = torch.from_numpy(np.asarray(slots, np.int64)).cuda()
        got = [_attend64(Q[h], torch.cat([K[h][at].reshape(-1, c["d"]), Kq[h]]),
                         torch.cat([V[h][at].reshape(-1, c["d"]), Vq[h]]), scale, c["F"]) for h in range(n)]
        O, lse, mass = (torch.stack(x) for x in zip(*got))
        return {"mass": mass, "O": O, "lse": lse}
    if c["kind"] == "score":
        scores, kept_seg, *_ = layer(K, V, slots, Q, Kq, Vq, attend=None)
        return {"scores": scores, "kept_seg": kept_seg, "kv_len": None}
    if c["kind"] == "compress":
        scores, kept_seg, rows, *_ = layer(K, V, slots, Q, Kq, Vq, attend=False)
        slab = max(_tokens(c, b) for b in heads)
        out = [torch.zeros((n, slab, c["d"]), dtype=torch.float64, device="cuda") for _ in range(2)]
        for h, kv in enumerate(rows):
            for x, r in zip(out, kv):
                x[h, :len(r)] = r.double()
        return {"Kc": out[0], "Vc": out[1], "scores": scores, "kept_seg": kept_seg, "kv_len": None}
    scores, kept_seg, _, O, lse = layer(K, V, slots, Q, Kq, Vq)
    out = {"O": torch.stack(O), "scores": scores, "kept_seg": kept_seg}
    if c["lse"]:
        out["lse"] = torch.stack(lse)
    return out
