"""The top-k reduction against a plain sum in 64 bits: every k with a kernel of its own and one without, with a number of tokens
that its groups of 1, 2 or 4 do not divide, on both sides of the size from which a group holds several tokens."""
import numpy as np
import pytest

import workloads as wl
from oracle import moe_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [3, 8191, 16387])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 8])
def test_tokens_that_do_not_fill_a_group(T, k):
    import gpu_harness as H
    cfg = wl.MoEConfig("combine", T=T, H=512, F=128, E=8, k=k, act=wl.ACT_SWIGLU, S=1, seed=740 + k)
    inp = wl.make_inputs(cfg, threads=4)
    ids, w = orc.route_topk(inp.logits, k)
    print(f"combine T {T} k {k}", flush=True)
    layer = H.GpuLayer(cfg, inp, ids, w)
    layer.out.fill_(7.0)
    layer.forward()
    run = layer.results()
    layer.close()
    assert run.status == 0
    rows = np.unique(np.concatenate([np.arange(min(T, 64)), np.arange(max(0, T - 64), T), np.random.default_rng(k).integers(0, T, 64)]))
    ref = orc.moe_layer(inp.x[rows], inp.W1, inp.W2, ids[rows], w[rows], cfg.act)
    a, b = H.error_metrics(run.out[rows], ref)
    assert a <= H.REL_TOL and b <= H.REL_TOL, f"{a:.3e} {b:.3e}"
    assert np.isfinite(run.out).all() and not (run.out == 7.0).all(axis=1).any()
