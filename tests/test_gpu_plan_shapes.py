"""Score reduction over the shapes at which its launch changes (workgroups of
64 or 32 positions, one or several groups of positions to a workgroup, one or
several passes over the frames) against the oracle.  The sums are float64 in
the oracle's order, rounded once to float32: core layers equal, Q, V and A
within the bounds of the other reduction tests."""
import numpy as np
import pytest
import torch

import oracle as O
import workload as W
from helpers import dev, host, maxrel, rowwise_maxrel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


@pytest.mark.parametrize("batch,layers,frames,n_s", [
    (1, 3, 17, 33), (2, 2, 33, 64), (1, 64, 64, 97),      # 32 positions, ragged; every frame count of a pass
    (64, 2, 64, 250), (3, 5, 16, 65), (1, 4, 1, 2),       # 64 positions, frames in several passes or one
    (64, 2, 16, 577), (40, 3, 20, 900), (64, 1, 3, 4096)])  # several groups of positions to a workgroup
def test_score_reduce_shapes(batch, layers, frames, n_s):
    from paper_2609_38984_amd import swam
    cfg = W.preset(1).replace(batch=batch, d_model=64, n_heads=1, n_blocks=layers, n_ctx=1, n_frames=frames,
                              frame_h=1, frame_w=n_s, n_act=frames, k_core=1, k_anchor=0)
    rng = np.random.default_rng(batch * 1000 + n_s)
    s = rng.gamma(0.3, 1.0, (batch, layers, frames, n_s)).astype(np.float32)
    ctx = swam.Context(cfg)
    k = min(cfg.k_layer, layers)
    v = torch.full((batch, frames, n_s), -1.0, device="cuda:0")
    a = torch.full((batch, n_s), -1.0, device="cuda:0")
    q = torch.full((batch, layers), -1.0, device="cuda:0")
    core = torch.full((batch, k), -1, dtype=torch.int32, device="cuda:0")
    ctx.score_reduce(dev(s), v, a, q, core)
    torch.cuda.synchronize()
    for b in range(batch):
        r = O.score_reduce(s[b], cfg.k_layer, cfg.cv_penalty)
        np.testing.assert_array_equal(host(core)[b], r.L_core)
        assert maxrel(host(q)[b], r.Q) < 1e-6
        assert rowwise_maxrel(host(v)[b], r.V) < 1e-5
        assert maxrel(host(a)[b], r.A) < 1e-5
