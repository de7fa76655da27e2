"""Degenerate cases of the step on the GPU against the oracle (fp32, outputs
1e-4 max-relative, selection bit-exact, pruned rows byte-identical): no
retained future token, no context, a single 7-token frame, two-token frames,
one action query per frame, a mass threshold of 1, the most blocks a model may
have (64: every layer scored, K_layer of 64 reduced), and a zero-row block."""
import numpy as np
import pytest
import torch

import oracle as O
import workload as W
from helpers import dev, host, maxrel, model_for

pytestmark = pytest.mark.gpu

BASE = W.preset(1)
CASES = {
    "no_future_token_kept": BASE.replace(k_core=0, k_anchor=0),
    "no_context": BASE.replace(n_ctx=0),
    "one_frame_of_7": BASE.replace(n_frames=1, frame_h=1, frame_w=7, n_act=4, k_core=3, k_anchor=2),
    "two_token_frames": BASE.replace(frame_h=1, frame_w=2, k_core=1, k_anchor=1),
    "one_query_per_frame": BASE.replace(n_act=2),
    "mass_threshold_one": BASE.replace(mass_threshold=1.0, k_core=64, k_anchor=0),
    "max_blocks": BASE.replace(n_blocks=64),
}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


@pytest.mark.parametrize("name", list(CASES))
def test_degenerate_schedule_matches_oracle(name):
    from paper_2609_38984_amd import swam
    cfg = CASES[name]
    print(f"edge case {name}: L_full={cfg.l_full} N_s={cfg.n_s} F={cfg.n_frames} H={cfg.n_act}",
          flush=True)
    blocks, _, model = model_for(cfg)
    inp = W.make_inputs(cfg, blocks[0]["w_qkv"])
    ys, refr = O.run_schedule(cfg, blocks, inp.x, inp.temb)
    ctx = swam.Context(cfg)
    for tau in range(cfg.n_steps):
        x = dev(inp.x(tau))
        y = torch.empty_like(x)
        kind = ctx.step(model, x, dev(inp.temb(tau)), tau, y)
        torch.cuda.synchronize()
        err = maxrel(host(y), ys[tau])
        print(f"  tau {tau} kind {kind} max-rel {err:.2e}", flush=True)
        assert err < 1e-4
        if tau in refr:
            pp = torch.empty(cfg.l_full, dtype=torch.int32, device="cuda:0")
            ctx.export(pack_pos=pp)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(pp.cpu().numpy(), refr[tau].packmap.pack_pos)
            assert ctx.packed_rows() == int(refr[tau].packmap.cu_seqlens[-1])
        else:
            pruned = refr[cfg.reuse_R * (tau // cfg.reuse_R)].packmap.pack_pos < 0
            assert y.cpu().numpy()[pruned].tobytes() == x.cpu().numpy()[pruned].tobytes()


def test_block_with_zero_rows_is_a_no_op():
    cfg = BASE
    _, dblocks, _ = model_for(cfg, 1)
    from paper_2609_38984_amd import swam
    ctx = swam.Context(cfg)
    x = torch.full((4, cfg.d_model), 3.0, device="cuda:0")
    cu = torch.zeros(2, dtype=torch.int32, device="cuda:0")
    ctx.block(dblocks[0], dev(W.timestep_embedding(cfg, 0)), x, 0, cu, 1)
    torch.cuda.synchronize()
    assert (x == 3.0).all()


def test_misaligned_tensors_are_rejected_before_any_launch():
    """The kernels move weights and activation rows in 16-byte vectors: a view
    4 bytes off its allocation must come back as SWAM_E_INVALID from the host
    checks, with nothing written."""
    from paper_2609_38984_amd import swam
    cfg = BASE
    _, dblocks, model = model_for(cfg)
    ctx = swam.Context(cfg)
    n = cfg.l_full * cfg.d_model
    buf = torch.zeros(2 * n + 8, dtype=torch.float32, device="cuda:0")
    x_ok = buf[:n].view(cfg.l_full, cfg.d_model)
    x_bad = buf[n + 1:2 * n + 1].view(cfg.l_full, cfg.d_model)
    temb = dev(W.timestep_embedding(cfg, 0))
    with pytest.raises(swam.SwamError) as e:
        ctx.block(dblocks[0], temb, x_bad)
    assert e.value.code == -1 and "aligned" in str(e.value)
    w_bad = dict(dblocks[0])
    wq = w_bad["w_qkv"]
    wbuf = torch.zeros(wq.numel() + 8, dtype=wq.dtype, device="cuda:0")
    w_bad["w_qkv"] = wbuf[1:1 + wq.numel()].view_as(wq)
    with pytest.raises(swam.SwamError) as e:
        ctx.block(w_bad, temb, x_ok)
    assert e.value.code == -1 and "aligned" in str(e.value)
    with pytest.raises(swam.SwamError) as e:
        ctx.step(model, x_ok, temb, 0, x_bad)
    assert e.value.code == -1 and "aligned" in str(e.value)
    torch.cuda.synchronize()
    assert bool((buf == 0).all())


def test_partially_overlapping_output_is_rejected():
    """y_full is x_full itself or disjoint from it (the pruned rows are copied
    and the retained ones scattered on that assumption): an output a few rows
    into the input must come back as SWAM_E_INVALID with nothing written."""
    from paper_2609_38984_amd import swam
    cfg = BASE
    _, _, model = model_for(cfg)
    ctx = swam.Context(cfg)
    n = cfg.l_full * cfg.d_model
    buf = torch.zeros(n + 4 * cfg.d_model, dtype=torch.float32, device="cuda:0")
    x = buf[:n].view(cfg.l_full, cfg.d_model)
    y = buf[4 * cfg.d_model:].view(cfg.l_full, cfg.d_model)
    temb = dev(W.timestep_embedding(cfg, 0))
    for a, b in ((x, y), (y, x)):
        with pytest.raises(swam.SwamError) as e:
            ctx.step(model, a, temb, 0, b)
        assert e.value.code == -1 and "overlap" in str(e.value)
    torch.cuda.synchronize()
    assert bool((buf == 0).all())


def test_exports_to_unaligned_buffers():
    """Exports into buffers that start between 16-byte boundaries (their copy
    then moves words) hold the bytes of the aligned ones, and nothing around
    them changes."""
    from paper_2609_38984_amd import swam
    cfg = BASE.replace(frame_h=3, frame_w=7, k_core=5, k_anchor=3)
    blocks, _, model = model_for(cfg)
    inp = W.make_inputs(cfg, blocks[0]["w_qkv"])
    ctx = swam.Context(cfg)
    x = dev(inp.x(0))
    ctx.step(model, x, dev(inp.temb(0)), 0, torch.empty_like(x))
    n_v, k = cfg.batch * cfg.n_frames * cfg.n_s, cfg.k_core + cfg.k_anchor
    sizes = dict(v=(n_v, torch.float32), a=(cfg.batch * cfg.n_s, torch.float32),
                 keep_idx=(cfg.batch * cfg.n_frames * k, torch.int32),
                 pack_pos=(cfg.batch * cfg.l_full, torch.int32), cu_seqlens=(cfg.batch + 1, torch.int32))
    want = {name: torch.full((n,), -7, dtype=t, device="cuda:0") for name, (n, t) in sizes.items()}
    ctx.export(**want)
    for off in (1, 2, 3):
        bufs = {name: torch.full((n + 8,), -7, dtype=t, device="cuda:0") for name, (n, t) in sizes.items()}
        ctx.export(**{name: b[off:off + sizes[name][0]] for name, b in bufs.items()})
        torch.cuda.synchronize()
        for name, b in bufs.items():
            n = sizes[name][0]
            assert torch.equal(b[off:off + n], want[name]), (name, off)
            assert bool((b[:off] == -7).all()) and bool((b[off + n:] == -7).all()), (name, off)
