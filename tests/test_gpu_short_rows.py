"""Projections of short token sets (the ring kernel, its K splits and the
LayerNorm that shares the pass summing them) on the GPU against the oracle:
row counts at the edges of the 64- and 128-row tiles, widths whose column
tiles are ragged, short and long K, one block at a time and as a chain of
blocks, with and without rotary embedding and QK-norm, in bf16 and fp32 (whose
projections all run that kernel, and whose attention splits the keys of 32
query rows over four waves).  Block outputs are held to the tolerances of every
block here: 2e-2 max-relative in bf16 (storage of the residual stream and of
every projection) and 1e-4 in fp32.  The shapes of the bf16 attention are
checked on the attention output and normaliser themselves."""
import numpy as np
import pytest
import torch

import oracle as O
import workload as W
from helpers import act_dtype, dev, host, maxrel, model_for

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def _cfg(heads, rows, **kw):
    # n_ctx + 1 frame of 2 + 1 action token = rows
    return W.preset(2).replace(d_model=64 * heads, n_heads=heads, n_blocks=1, n_ctx=max(rows - 3, 0), n_frames=1,
                               frame_h=1, frame_w=2, n_act=1, k_core=1, k_anchor=0, **kw)


TOL = {"bf16": 2e-2, "f32": 1e-4}


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("variant", [dict(), dict(rope=1, qk_norm=1)])
@pytest.mark.parametrize("heads,rows", [(1, 3), (1, 64), (2, 65), (3, 127), (5, 129), (8, 192), (7, 193), (17, 321),
                                        (24, 192), (12, 700), (5, 2049)])   # (the last: QKV on 128x64 tiles)
def test_block_short_rows(heads, rows, variant, dtype):
    from paper_2609_38984_amd import swam
    cfg = _cfg(heads, rows, dtype=dtype, **variant)
    blocks, dblocks, _ = model_for(cfg, 1)
    x = W.make_inputs(cfg, blocks[0]["w_qkv"]).x(0)
    temb = W.timestep_embedding(cfg, 0)
    # two sequences of unequal length
    cu = np.array([0, rows // 3, rows], np.int32)
    pos = np.concatenate([np.arange(rows // 3), np.arange(rows - rows // 3)])
    want, _ = O.block(x, blocks[0], temb, cu, heads, cfg.dtype, positions=pos, rope=bool(cfg.rope),
                      qk_norm=bool(cfg.qk_norm))
    ctx = swam.Context(cfg)
    y = dev(x, act_dtype(cfg))
    print(f"block of {heads} heads, {rows} rows {variant}", flush=True)
    ctx.block(dblocks[0], dev(temb), y, rows, dev(cu), 2)
    torch.cuda.synchronize()
    err = maxrel(host(y), want)
    print(f"  max-rel {err:.2e}", flush=True)
    assert err < TOL[dtype]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("heads,rows", [(1, 70), (9, 130), (24, 192), (33, 100), (9, 1151), (3, 2689), (11, 2689)])
def test_step_chains_the_layer_norms(heads, rows, dtype):
    """Dense steps of 3 blocks: the next block's first LayerNorm comes out of
    the pass that sums the split down projection (33 heads: two chunks of a row
    per thread there).  The last three run 128x64 tiles at the edges of 128
    rows: split down projections in bf16 (9 heads) and fp32 (3 heads), a split
    out projection in fp32 (9 heads), out and down without a split in both (11
    heads)."""
    from paper_2609_38984_amd import swam
    cfg = _cfg(heads, rows, dtype=dtype).replace(n_blocks=3)
    blocks, _, model = model_for(cfg)
    inp = W.make_inputs(cfg, blocks[0]["w_qkv"])
    want = O.dense_step(inp.x(0), blocks, inp.temb(0), cfg)
    ctx = swam.Context(cfg)
    x = dev(inp.x(0), act_dtype(cfg))
    y = torch.empty_like(x)
    print(f"step of {heads} heads, {rows} rows", flush=True)
    ctx.step(model, x, dev(inp.temb(0)), 0, y, swam.FORCE_DENSE)
    torch.cuda.synchronize()
    err = maxrel(host(y), want)
    print(f"  max-rel {err:.2e}", flush=True)
    assert err < TOL[dtype]


@pytest.mark.parametrize("heads,cu", [
    (4, [0, 1, 1, 2]), (8, [0, 63, 128, 193]), (1, [0, 65]), (12, [0, 1312]),   # 64-row tiles, keys split
    (16, [0, 1312]), (16, [0, 384, 384, 1153]), (12, [0, 130, 1500]),           # 128-row tiles, keys split
    (16, [0, 200, 200, 330, 1100]), (20, [0, 600, 1300, 1999]),                 # 128-row tiles
    (16, [0, 1312, 2500]), (13, [0, 2561])])                                    # 256-row tiles
def test_block_attention_shapes(heads, cu):
    """Every shape the bf16 attention is dispatched in, with sequences shorter
    than a tile of keys, empty ones and lengths at the edges of the tiles.

    Logits of standard deviation 3 put most of a row's weight on a few keys
    anywhere in its sequence, and an identity output projection behind a gate
    of 64 with the MLP's gate at 0 shows the attention output itself.  The
    normaliser and the output are checked from the kernel's own q, k and v.
    The bound: bf16 has 8 significant bits, so rounding to nearest errs by up to
    2^-8 of a value; the probabilities are rounded (2^-8 of sum p |v|), the
    output is stored (2^-8 of |o|) and so is y = x + 64 o (2^-8 of |o| + |x| /
    64); 1% and 1e-4 of sum p |v| for the fp32 sums and exponentials.  A reference that
    leaves out one key of each sequence exceeds it many times over."""
    from paper_2609_38984_amd import swam
    rows, d = cu[-1], 64 * heads
    cfg = _cfg(heads, max(rows, 3), dtype="bf16")
    rng = np.random.default_rng(rows + heads)
    w = W.block_weights(cfg, 0)
    w["w_ada"] = np.zeros_like(w["w_ada"])
    w["b_ada"] = np.repeat(np.array([0, 0, 64, 0, 0, 0], np.float32), d)
    w["w_qkv"][:2 * d] = O.round_bf16(w["w_qkv"][:2 * d] * 3.0 ** 0.5)
    w["w_o"] = np.eye(d, dtype=np.float32)
    w["b_o"] = np.zeros_like(w["b_o"])
    x = O.round_bf16(rng.standard_normal((rows, d)))
    dw = {k: dev(v, torch.bfloat16) for k, v in w.items()}
    ctx = swam.Context(cfg)
    y = dev(x, torch.bfloat16)
    lse = torch.full((rows, heads), 7.0, device="cuda:0")
    qkv = torch.empty((rows, 3 * d), dtype=torch.bfloat16, device="cuda:0")
    print(f"attention of {heads} heads, sequences {cu}", flush=True)
    ctx.block(dw, dev(W.timestep_embedding(cfg, 0)), y, rows, dev(np.array(cu, np.int32)), len(cu) - 1, lse, qkv)
    torch.cuda.synchronize()
    q, k, v = np.split(host(qkv).reshape(rows, 3, heads, 64), 3, axis=1)
    got, lam, x = (host(y) - x).reshape(rows, heads, 64) / 64.0, host(lse), x.reshape(rows, heads, 64)
    worst, planted = 0.0, np.inf
    for a, b in zip(cu[:-1], cu[1:]):
        if a == b:
            continue
        without = 0.0
        for h in range(heads):
            logit = q[a:b, 0, h] @ k[a:b, 0, h].T / 8.0
            top = logit.max(axis=1, keepdims=True)
            e = np.exp(logit - top)
            total = e.sum(axis=1, keepdims=True)
            want_lam = (top + np.log(total))[:, 0]
            assert (np.abs(lam[a:b, h] - want_lam) / np.maximum(1.0, np.abs(want_lam))).max() < 1e-5
            vh = v[a:b, 0, h]
            o, mass = e @ vh / total, e @ np.abs(vh) / total
            bound = 2.0 ** -8 * 1.01 * (mass + 2.0 * np.abs(o) + np.abs(x[a:b, h]) / 64.0) + 1e-4 * mass
            worst = max(worst, (np.abs(got[a:b, h] - o) / bound).max())
            if b - a > 1:                        # the last key left out
                part = e[:, :-1] @ vh[:-1] / e[:, :-1].sum(axis=1, keepdims=True)
                without = max(without, (np.abs(part - o) / bound).max())
        if b - a > 1:
            planted = min(planted, without)
    print(f"  error {worst:.2f} of the bound, a lost key {planted:.0f}", flush=True)
    assert worst <= 1.0
    assert planted > 10.0 or rows <= 2
