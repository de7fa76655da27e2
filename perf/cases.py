"""Performance cases of the action-guided sparse denoising step.

Each case is one call (or the few calls) that a sampling program makes on this
framework, through `paper_2609_38984_amd.swam`: a dense, refresh or sparse
step of the block stack, a whole closed-loop sampling step, or the score
reduction with the selection that follows it.  Sizes are those of the
repository's own workloads (`workload/`, `bench.py`), or drawn around them.

`prepare` makes what such a program holds before the call (weights, tokens,
the context with its workspace, a cached selection), `run` is one pass,
`exact` the same result in float64 by plain torch.
"""
import math
import types

import torch

from paper_2609_38984_amd import swam

HEAD = 64
D_TEMB = 128


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def _case(**kw):
    case = dict(kind="step", phase="dense", dtype="bf16", batch=1, heads=24, blocks=1, n_ctx=98,
                frames=2, h=1, w=98, n_act=32, k_core=19, k_anchor=12, ragged=False, rope=0,
                qk_norm=0, pairs=0, guidance=1.0, graph=False, d_latent=0)
    case.update(kw)
    return case


_WAM = dict(heads=24, n_ctx=512, frames=8, h=30, w=40, n_act=48, k_core=300, k_anchor=64)
_D2048 = dict(heads=32, n_ctx=1024, frames=16, h=32, w=32, n_act=64, k_core=256, k_anchor=64)
_RAGGED = dict(batch=8, heads=24, n_ctx=256, frames=4, h=24, w=32, n_act=32, k_core=768, k_anchor=0)
_VIEW3 = dict(batch=2, heads=24, n_ctx=340, frames=8, h=1, w=340, n_act=32, k_core=80, k_anchor=104)


def listed():
    return [
        # the smallest call: a debug / unit-size policy in float32, one refresh; launches and latency
        _case(name="tiny_f32_refresh", phase="refresh", dtype="f32", heads=2, n_ctx=16, frames=2,
              h=8, w=8, n_act=8, k_core=16, k_anchor=4),
        # float32 at a real width: the check run of a policy before it is put to bf16 (2 views, 98 tokens)
        _case(name="view2_f32_sparse_2blk", phase="sparse", dtype="f32", blocks=2),
        # the sparse step of a 30-layer robot policy at batch 1, replayed as a graph: 9 of its 10 steps
        _case(name="view2_sparse_30blk_graph", phase="sparse", blocks=30, graph=True),
        # the same policy's full step, enqueued launch by launch
        _case(name="view2_dense_30blk", phase="dense", blocks=30),
        # a mid-size model's full step with scoring and selection
        _case(name="d1024_refresh_2blk", phase="refresh", heads=16, blocks=2, n_ctx=256, frames=4,
              h=16, w=16, n_act=32, k_core=77, k_anchor=16),
        # closed-loop sampling step of a guided 3-camera policy with rotary q / k and QK-norm
        _case(name="view3_cfg_sample_sparse_2blk", kind="sample", phase="sparse", blocks=2, rope=1,
              qk_norm=1, pairs=1, guidance=3.0, d_latent=16, **_VIEW3),
        # the benchmark's world-action model: full step with scoring and selection, then the sparse step
        _case(name="wam_refresh_2blk", phase="refresh", blocks=2, **_WAM),
        _case(name="wam_sparse_2blk", phase="sparse", blocks=2, **_WAM),
        # the largest: d = 2048, 17,472 tokens, full and sparse
        _case(name="d2048_dense_1blk", phase="dense", **_D2048),
        _case(name="d2048_sparse_2blk", phase="sparse", blocks=2, **_D2048),
        # a serving batch of 8 sequences of unequal retained length
        _case(name="ragged_b8_sparse_1blk", phase="sparse", ragged=True, **_RAGGED),
        # score reduction and selection on the scores of 28 layers (the part between two steps)
        _case(name="wam_plan_28layers", kind="plan", phase="plan", blocks=28, **_WAM),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    largest = work(listed()[8])["flops"]
    while True:
        kind = rng.choice(["dense", "dense", "refresh", "refresh", "sparse", "sparse", "sparse", "sample",
                           "plan", "f32"])
        frames = rng.choice([1, 2, 3, 4, 6, 8, 12, 16])
        n_s = _log_int(rng, 48, 1300)
        batch = rng.choice([1, 1, 1, 1, 2, 3, 8])
        k_core = max(1, int(n_s * rng.uniform(0.12, 0.4)))
        c = _case(kind="step", batch=batch, heads=_log_int(rng, 6, 32), blocks=rng.choice([1, 2]),
                  n_ctx=_log_int(rng, 40, 1100), frames=frames, h=1, w=n_s,
                  n_act=frames * rng.randint(1, 16), k_core=k_core,
                  k_anchor=int((n_s - k_core) * rng.uniform(0.0, 0.35)),
                  rope=rng.choice([0, 0, 1]), qk_norm=rng.choice([0, 0, 1]), graph=rng.choice([False, True]))
        if kind in ("dense", "refresh", "sparse"):
            c.update(phase=kind)
            if kind == "sparse" and batch > 1 and rng.random() < 0.5:
                c.update(ragged=True, k_core=n_s, k_anchor=0)
        elif kind == "sample":
            c.update(kind="sample", phase=rng.choice(["dense", "sparse"]), d_latent=rng.choice([8, 16, 24, 48]),
                     graph=False)
            if batch % 2 == 0:
                c.update(pairs=1, guidance=3.0)
        elif kind == "plan":
            c.update(kind="plan", phase="plan", blocks=rng.randint(6, 36), rope=0, qk_norm=0, graph=False)
        else:
            c.update(dtype="f32", phase=rng.choice(["dense", "refresh", "sparse"]), batch=1, frames=rng.choice([1, 2, 4]),
                     heads=_log_int(rng, 2, 24), w=_log_int(rng, 40, 128), n_ctx=_log_int(rng, 16, 128))
            n_s = c["w"]
            c.update(n_act=c["frames"] * rng.randint(1, 16), k_core=max(1, int(n_s * rng.uniform(0.12, 0.4))))
            c.update(k_anchor=int((n_s - c["k_core"]) * rng.uniform(0.0, 0.35)))
        if work(c)["flops"] <= largest:
            return c


# ---------------------------------------------------------------------------
# sizes
# ---------------------------------------------------------------------------
def _sizes(case):
    n_s = case["h"] * case["w"]
    l_full = case["n_ctx"] + case["frames"] * n_s + case["n_act"]
    scored = case["batch"] // 2 if case["pairs"] else case["batch"]
    return n_s, l_full, scored, case["heads"] * HEAD


def _config(case):
    return types.SimpleNamespace(
        batch=case["batch"], d_model=case["heads"] * HEAD, n_heads=case["heads"], head_dim=HEAD,
        mlp_ratio=4, n_blocks=case["blocks"], d_temb=D_TEMB, n_ctx=case["n_ctx"],
        n_frames=case["frames"], frame_h=case["h"], frame_w=case["w"], n_act=case["n_act"],
        k_core=case["k_core"], k_anchor=case["k_anchor"], k_layer=6, cv_penalty=1.0,
        mass_threshold=0.8 if case["ragged"] else 0.0, reuse_R=4, dtype=case["dtype"],
        rope=case["rope"], qk_norm=case["qk_norm"], cfg_pairs=case["pairs"], guidance=case["guidance"])


def _counts(case):
    """Retained tokens of every sequence and frame ([B][F]); ragged batches keep
    between 20% and 60% of a frame, as a score-mass threshold does."""
    n_s, _, scored, _ = _sizes(case)
    if not case["ragged"]:
        return [[case["k_core"] + case["k_anchor"]] * case["frames"]] * case["batch"]
    one = [[max(1, int(n_s * (0.2 + 0.4 * ((7 * b + 3 * f) % 11) / 10))) for f in range(case["frames"])]
           for b in range(scored)]
    return one * 2 if case["pairs"] else one


def _lengths(case):
    _, l_full, _, _ = _sizes(case)
    if case["phase"] != "sparse":
        return [l_full] * case["batch"]
    return [case["n_ctx"] + sum(c) + case["n_act"] for c in _counts(case)]


def work(case):
    """One pass: every weight read once, the tokens read and written once, the
    projections and the attention of the rows that are computed."""
    n_s, l_full, scored, d = _sizes(case)
    es = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "plan":
        maps = scored * case["frames"] * n_s
        kept = sum(sum(c) for c in _counts(case)[:scored])
        rows = case["batch"] * l_full
        return {"bytes": 4.0 * (case["blocks"] * maps + maps + scored * n_s + kept + 2 * rows),
                "flops": 4.0 * case["blocks"] * maps}
    lens = _lengths(case)
    rows = sum(lens)
    per_block = 12 * d * d + 9 * d + 6 * d * (D_TEMB + 1)
    flops = case["blocks"] * (24.0 * rows * d * d + 4.0 * d * sum(n * n for n in lens) + 12.0 * d * D_TEMB)
    nbytes = float(es) * case["blocks"] * per_block + 2.0 * es * case["batch"] * l_full * d
    if case["phase"] == "refresh":
        flops += case["blocks"] * 2.0 * scored * case["n_act"] * n_s * d
        nbytes += 4.0 * scored * n_s * (case["frames"] + 1)
    if case["kind"] == "sample":
        lat = case["frames"] * n_s + case["n_act"]
        c = case["d_latent"]
        flops += 4.0 * case["batch"] * lat * c * d
        nbytes += 4.0 * lat * c * (4 * scored + case["batch"]) + 2.0 * es * c * d
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["kind"] == "plan":
        # float64 sums rounded once to float32; a last bit may move one tie of the order
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.002}
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 2e-4}
    if case["blocks"] > 4:
        return {"rel": 0.03, "max": 0.5}
    return {"rel": 0.015, "max": 0.25}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
_WEIGHTS = (("w_ada", lambda d: (6 * d, D_TEMB)), ("b_ada", lambda d: (6 * d,)),
            ("w_qkv", lambda d: (3 * d, d)), ("b_qkv", lambda d: (3 * d,)),
            ("w_o", lambda d: (d, d)), ("b_o", lambda d: (d,)),
            ("w_1", lambda d: (4 * d, d)), ("b_1", lambda d: (4 * d,)),
            ("w_2", lambda d: (d, 4 * d)), ("b_2", lambda d: (d,)))


def _inputs(case, seed):
    """Tensors of a case from its seed: weights N(0, 1 / fan_in), unit tokens
    with one action-relevant blob per frame, the timestep embedding, and a
    selection of the cached budget."""
    g = torch.Generator(device="cuda").manual_seed(0x5EED + int(seed))
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    n_s, l_full, scored, d = _sizes(case)
    b, f = case["batch"], case["frames"]

    def normal(shape, std=1.0, dtype=dt):
        return torch.randn(shape, device="cuda", generator=g).mul_(std).to(dtype)

    s = types.SimpleNamespace()
    if case["kind"] == "plan":
        # scores fall off over orders of magnitude, as softmax weights do
        s.s_all = torch.exp(normal((scored, case["blocks"], f, n_s), 1.5, torch.float32) - 8.0)
        return s
    s.blocks = []
    for _ in range(case["blocks"]):
        w = {}
        for name, shape in _WEIGHTS:
            fan = D_TEMB if "ada" in name else 4 * d if name.endswith("_2") else d
            w[name] = normal(shape(d), fan ** -0.5)
        s.blocks.append(w)
    t = 1000.0 * float(torch.rand((), device="cuda", generator=g))
    freq = torch.exp(-math.log(10000.0) * torch.arange(D_TEMB // 2, dtype=torch.float64) / (D_TEMB // 2))
    s.temb = torch.cat([torch.cos(t * freq), torch.sin(t * freq)]).float().cuda()
    x = normal((b, l_full, d), 1.0, torch.float32)
    act = x[:, l_full - case["n_act"]:]
    # token direction that raises the logits of each frame's own action queries
    wq, wk = s.blocks[0]["w_qkv"][:d].float(), s.blocks[0]["w_qkv"][d:2 * d].float()
    mean = act.reshape(b, f, -1, d).mean(2).reshape(b * f, d)
    u = (mean @ wq.t().contiguous()) @ wk
    u = (u * (d ** 0.5 / u.norm(dim=1, keepdim=True))).reshape(b, f, 1, d)
    at = torch.arange(n_s, device="cuda", dtype=torch.float32)
    centre = torch.rand((b, f, 1, 1), device="cuda", generator=g) * n_s
    blob = torch.exp(-((at.reshape(1, 1, n_s, 1) - centre) / max(2.0, n_s / 20)) ** 2 / 2)
    x[:, case["n_ctx"]:l_full - case["n_act"]] += (0.5 * blob * u).reshape(b, f * n_s, d)
    s.x = x.to(dt).reshape(b * l_full, d).contiguous()
    # retained positions: the highest of random keys, ascending, padded with -1
    counts = torch.tensor(_counts(case)[:scored], device="cuda")
    order = torch.rand((scored, f, n_s), device="cuda", generator=g).argsort(-1).argsort(-1)
    s.kept = order < counts.reshape(scored, f, 1)
    if case["pairs"]:
        s.kept = torch.cat([s.kept, s.kept])
    if case["kind"] == "sample":
        c, lat = case["d_latent"], f * n_s + case["n_act"]
        s.io = {"w_in": normal((d, c), c ** -0.5), "b_in": normal((d,), c ** -0.5),
                "w_v": normal((c, d), d ** -0.5), "b_v": normal((c,), d ** -0.5)}
        s.z0 = normal((scored * lat, c), 1.0, torch.float32)
        s.v_cache = normal((scored * lat, c), 1.0, torch.float32)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s.case = case
    n_s, l_full, scored, d = _sizes(case)
    # a graph is captured on a stream of the program's own
    s.stream = torch.cuda.Stream() if case["graph"] else None
    s.ctx = swam.Context(_config(case), s.stream)
    if case["kind"] == "plan":
        dev = dict(device="cuda")
        s.v = torch.empty((scored, case["frames"], n_s), **dev)
        s.a = torch.empty((scored, n_s), **dev)
        s.q = torch.empty((scored, case["blocks"]), **dev)
        rows, k_max = case["batch"] * l_full, s.ctx.k_max
        s.keep_idx = torch.zeros((case["batch"], case["frames"], k_max), dtype=torch.int32, **dev)
        s.keep_cnt = torch.zeros((case["batch"], case["frames"]), dtype=torch.int32, **dev)
        s.pack_pos = torch.zeros(rows, dtype=torch.int32, **dev)
        s.gather = torch.zeros(rows, dtype=torch.int32, **dev)
        s.cu = torch.zeros(case["batch"] + 1, dtype=torch.int32, **dev)
        return s
    s.model = swam.Model(s.blocks, s.x.dtype)
    s.y = torch.empty_like(s.x)
    if case["phase"] == "sparse":
        k_max = s.ctx.k_max
        at = torch.where(s.kept, torch.arange(n_s, device="cuda"), n_s).sort(-1).values[..., :k_max]
        idx = torch.where(at < n_s, at, -1).to(torch.int32).contiguous()
        torch.cuda.synchronize()
        s.ctx.set_selection(idx)
    if case["phase"] == "refresh":
        s.v = torch.empty((scored, case["frames"], n_s), device="cuda")
        s.a = torch.empty((scored, n_s), device="cuda")
    if case["kind"] == "sample":
        s.latent = swam.LatentIO(s.io, s.x.dtype)
        s.z = s.z0.clone()
        s.vel = torch.zeros((case["batch"] * (l_full - case["n_ctx"]), case["d_latent"]), device="cuda")
    return s


_FLAGS = {"dense": swam.FORCE_DENSE, "refresh": swam.FORCE_REFRESH, "sparse": 0}
_DSIGMA = -0.125


def run(s):
    case = s.case
    if case["kind"] == "plan":
        s.ctx.score_reduce(s.s_all, s.v, s.a, q_out=s.q)
        s.ctx.select(keep_idx=s.keep_idx, keep_cnt=s.keep_cnt, pack_pos=s.pack_pos, gather=s.gather,
                     cu_seqlens=s.cu)
        kept = case["batch"] * (case["n_ctx"] + case["frames"] * (case["k_core"] + case["k_anchor"]) + case["n_act"])
        return {"q": s.q, "v": s.v, "a": s.a, "keep_idx": s.keep_idx, "keep_cnt": s.keep_cnt,
                "pack_pos": s.pack_pos, "gather": s.gather[:kept], "cu": s.cu}
    flags = _FLAGS[case["phase"]]
    if case["kind"] == "sample":
        s.z.copy_(s.z0)
        s.ctx.sample_step(s.model, s.latent, s.z, s.vel, s.v_cache, s.x, s.y, s.temb, 1, _DSIGMA, flags)
        return {"z": s.z, "vel": s.vel, "y": s.y}
    if s.stream is not None:
        s.stream.wait_stream(torch.cuda.current_stream())
        s.ctx.step_graph(s.model, s.x, s.temb, 1, s.y, flags)
    else:
        s.ctx.step(s.model, s.x, s.temb, 1, s.y, flags)
    out = {"y": s.y}
    if case["phase"] == "refresh":
        s.ctx.export(v=s.v, a=s.a)
        out.update(v=s.v, a=s.a)
    if s.stream is not None:
        torch.cuda.current_stream().wait_stream(s.stream)
    return out


# ---------------------------------------------------------------------------
# the same in float64
# ---------------------------------------------------------------------------
def _norm(x, eps=1e-6):
    return (x - x.mean(-1, keepdim=True)) / torch.sqrt(x.var(-1, unbiased=False, keepdim=True) + eps)


def _block64(x, w, temb, lens, pos, case):
    """One block on concatenated sequences; returns the rows and q, k and the
    normaliser of every head."""
    d, heads = x.shape[1], case["heads"]
    mod = (w["w_ada"] @ (temb * torch.sigmoid(temb)) + w["b_ada"]).reshape(6, d)
    qkv = (_norm(x) * (1 + mod[1]) + mod[0]) @ w["w_qkv"].t() + w["b_qkv"]
    q, k, v = (t.reshape(-1, heads, HEAD) for t in qkv.split(d, 1))
    if case["qk_norm"]:
        q, k = (t / torch.sqrt(t.square().mean(-1, keepdim=True) + 1e-6) for t in (q, k))
    if case["rope"]:
        i = torch.arange(HEAD // 2, device=x.device, dtype=torch.float64)
        ang = (pos.double()[:, None] * 10000.0 ** (-2.0 * i / HEAD))[:, None, :]
        co, si = torch.cos(ang), torch.sin(ang)

        def turn(t):
            a, b = t[..., 0::2], t[..., 1::2]
            return torch.stack([a * co - b * si, a * si + b * co], -1).reshape(t.shape)
        q, k = turn(q), turn(k)
    o = torch.empty_like(q)
    lse = torch.empty(q.shape[:2], device=x.device, dtype=torch.float64)
    at = 0
    for n in lens:
        for h in range(heads):
            for r in range(at, at + n, 4096):
                e = min(at + n, r + 4096)
                logit = (q[r:e, h] / 8.0) @ k[at:at + n, h].t()
                lse[r:e, h] = torch.logsumexp(logit, 1)
                o[r:e, h] = torch.exp(logit - lse[r:e, h, None]) @ v[at:at + n, h]
        at += n
    x = x + mod[2] * (o.reshape(-1, d) @ w["w_o"].t() + w["b_o"])
    u = (_norm(x) * (1 + mod[4]) + mod[3]) @ w["w_1"].t() + w["b_1"]
    u = 0.5 * u * (1 + torch.tanh(math.sqrt(2 / math.pi) * (u + 0.044715 * u ** 3)))
    return x + mod[5] * (u @ w["w_2"].t() + w["b_2"]), q, k, lse


def _alpha(g):
    w = torch.tensor([2.0 if abs(i - (g - 1) / 2) < g / 4 else 1.0 for i in range(g)],
                     dtype=torch.float64, device="cuda")
    return w / w.sum()


def _plan64(s_all, n_s, k_layer=6):
    """Q, V and A of scores [B][L][F][N_s]."""
    mass = s_all.sum(-1)
    p = s_all / mass.clamp_min(1e-300)[..., None]
    ent = -(torch.where(p > 0, p * torch.log(p.clamp_min(1e-300)), torch.zeros_like(p))).sum(-1)
    frames = s_all.shape[2]
    q = mass.sum(-1) / frames * (1 - ent.sum(-1) / (frames * math.log(n_s)))
    core = q.topk(min(k_layer, q.shape[1]), dim=1).indices
    pick = torch.zeros_like(q).scatter_(1, core, 1.0) * q
    v = (pick[:, :, None, None] * s_all).sum(1) / pick.sum(1)[:, None, None]
    every = (q[:, :, None, None] * s_all).sum(1) / q.sum(1)[:, None, None]
    mu = every.mean(1)
    return q, v, mu / (1 + torch.sqrt(every.var(1, unbiased=False)) / mu)


def exact(case, seed):
    s = _inputs(case, seed)
    n_s, l_full, scored, d = _sizes(case)
    if case["kind"] == "plan":
        q, v, a = _plan64(s.s_all.double(), n_s)
        return {"q": q, "v": v, "a": a, "keep_idx": None, "keep_cnt": None, "pack_pos": None, "gather": None,
                "cu": None}
    b, f, n_ctx, n_act = case["batch"], case["frames"], case["n_ctx"], case["n_act"]
    temb = s.temb.double()
    x = s.x.double().reshape(b, l_full, d)
    if case["kind"] == "sample":
        tok = (s.z0.double() @ s.io["w_in"].double().t() + s.io["b_in"].double()).reshape(scored, -1, d)
        x[:, n_ctx:] = torch.cat([tok, tok]) if case["pairs"] else tok
    x = x.reshape(b * l_full, d)
    keep = torch.ones((b, l_full), dtype=torch.bool, device="cuda")
    if case["phase"] == "sparse":
        keep[:, n_ctx:l_full - n_act] = s.kept.reshape(b, f * n_s)
    rows = keep.reshape(-1).nonzero().reshape(-1)
    lens, pos, h = _lengths(case), rows % l_full, x[rows]
    maps = []
    for w in s.blocks:
        h, q, k, lse = _block64(h, {n: t.double() for n, t in w.items()}, temb, lens, pos, case)
        if case["phase"] == "refresh":
            g = n_act // f
            q, k, lse = (t.reshape(b, l_full, case["heads"], -1)[:scored] for t in (q, k, lse))
            qa = q[:, l_full - n_act:].reshape(scored, f, g, case["heads"], HEAD)
            la = lse[:, l_full - n_act:].reshape(scored, f, g, case["heads"])
            kf = k[:, n_ctx:l_full - n_act].reshape(scored, f, n_s, case["heads"], HEAD)
            score = torch.zeros((scored, f, n_s), dtype=torch.float64, device="cuda")
            for i, al in enumerate(_alpha(g).tolist()):
                logit = (qa[:, :, i, None] * kf).sum(-1) / 8.0 - la[:, :, i, None]
                score += al * torch.exp(logit).mean(-1)
            maps.append(score)
    y = x.clone()
    y[rows] = h
    if case["phase"] == "refresh":
        _, v, a = _plan64(torch.stack(maps, 1), n_s)
        return {"y": y, "v": v, "a": a}
    if case["kind"] != "sample":
        return {"y": y}
    vel = _norm(y.reshape(b, l_full, d)[:, n_ctx:]) @ s.io["w_v"].double().t() + s.io["b_v"].double()
    live = keep[:, n_ctx:, None]
    vel = vel * live
    step = vel[scored:] + case["guidance"] * (vel[:scored] - vel[scored:]) if case["pairs"] else vel
    if case["phase"] == "sparse":
        step = torch.where(live[:scored], step, s.v_cache.double().reshape(step.shape))
    z = s.z0.double() + _DSIGMA * step.reshape(s.z0.shape)
    return {"z": z, "vel": vel.reshape(-1, case["d_latent"]), "y": y}
