"""The tile kernel against the oracle at the edges of its tiles: experts with one row, with one row less and more than the
16-row blocks of an epilogue, than the 64-, 128- and 256-row tiles; every tile height, reductions of as few K steps as a
tile can have and of an even and an odd number of K step pairs; packed and plain weights, both activations."""
import numpy as np
import pytest

import workloads as wl
from oracle import moe_oracle as orc

pytestmark = pytest.mark.gpu

ROWS = (1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 193, 255, 256, 257, 0, 321)


@pytest.mark.parametrize("packed", [False, True], ids=["plain", "packed"])
@pytest.mark.parametrize("H,F,act", [(256, 128, wl.ACT_SWIGLU), (512, 384, wl.ACT_SWIGLU), (256, 256, wl.ACT_GELU)],
                         ids=["shortest", "odd", "gelu"])
def test_tile_edges(H, F, act, packed):
    import gpu_harness as G
    cfg = wl.MoEConfig("edges", T=sum(ROWS), H=H, F=F, E=len(ROWS), k=1, act=act, S=3, seed=720 + F)
    inp = wl.make_inputs(cfg, threads=4)
    ids = np.repeat(np.arange(cfg.E, dtype=np.int32), ROWS)[np.random.default_rng(7).permutation(cfg.T)][:, None].copy()
    w = np.linspace(0.5, 1.5, cfg.T, dtype=np.float32)[:, None].copy()
    ref = orc.moe_layer(inp.x, inp.W1, inp.W2, ids, w, act)
    for tile_m in (64, 128, 256):
        print(f"edges H {H} F {F} tile_m {tile_m} packed {packed}", flush=True)
        layer = G.GpuLayer(cfg, inp, ids, w, {"tile_m": tile_m}, packed=packed)
        layer.forward()
        run = layer.results()
        layer.close()
        assert run.status == 0
        a, b = G.error_metrics(run.out, ref)
        assert a <= G.REL_TOL and b <= G.REL_TOL, f"tile_m {tile_m}: {a:.3e} {b:.3e}"
