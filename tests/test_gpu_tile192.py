"""Tiles of 129 to 192 rows (the 192-row variant): alone and as the remainder beside full tiles, of one row more and less than
its ends and its 16-row blocks, among tiles of every other variant, with reductions of as few K steps as a tile can have and
more; packed and plain weights, both activations, the three places of the top-k reduction, one launch for both layers."""
import numpy as np
import pytest

import workloads as wl
from oracle import moe_oracle as orc

pytestmark = pytest.mark.gpu

ROWS = (129, 143, 144, 145, 160, 176, 177, 191, 192, 193, 128, 64, 256 + 129, 256 + 192, 512 + 150, 256, 0, 1, 170, 170)


@pytest.mark.parametrize("packed", [False, True], ids=["plain", "packed"])
@pytest.mark.parametrize("H,F,act", [(256, 128, wl.ACT_SWIGLU), (512, 384, wl.ACT_SWIGLU), (256, 768, wl.ACT_GELU)],
                         ids=["shortest", "odd", "gelu"])
def test_tiles_of_up_to_192_rows(H, F, act, packed):
    import gpu_harness as G
    cfg = wl.MoEConfig("tile192", T=sum(ROWS), H=H, F=F, E=len(ROWS), k=1, act=act, S=3, seed=900 + F)
    inp = wl.make_inputs(cfg, threads=4)
    ids = np.repeat(np.arange(cfg.E, dtype=np.int32), ROWS)[np.random.default_rng(9).permutation(cfg.T)][:, None].copy()
    w = np.linspace(0.5, 1.5, cfg.T, dtype=np.float32)[:, None].copy()
    ref = orc.moe_layer(inp.x, inp.W1, inp.W2, ids, w, act)
    first = None
    for options in ({}, {"n_cu": 8}, {"layer1_order": 1}, {"layer1_order": 2}, {"fuse_layers": 1}, {"tile_m": 128}):
        print(f"192-row tiles H {H} F {F} packed {packed} {options}", flush=True)
        layer = G.GpuLayer(cfg, inp, ids, w, {"tile_m": 256, **options}, packed=packed)
        layer.out.fill_(7.0)
        layer.forward()
        run = layer.results()
        layer.close()
        assert run.status == 0
        if first is None:
            first = run.out
            a, b = G.error_metrics(first, ref)
            assert a <= G.REL_TOL and b <= G.REL_TOL, f"{a:.3e} {b:.3e}"
        np.testing.assert_array_equal(run.out, first)
