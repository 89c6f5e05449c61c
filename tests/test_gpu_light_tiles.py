"""Remainders of an expert's rows beside its full tiles: tables and schedules where the light ones lie in the blocks of the full
ones in both layers, in one, and in none (where is checked per layer: beside from 128 items of them on, of experts of one block, and only
in the locality orders); few tiles and many (two ways to sort them); beside experts whose only tile is 64 or
128 rows high; with waves of source segments; tile heights of 128 and 256.  Table and schedules keep their invariants and the
outputs are the oracle's, with the same bits whatever the tile height."""
import numpy as np
import pytest

import workloads as wl
from oracle import moe_oracle as orc

pytestmark = pytest.mark.gpu

FULL_AND_LIGHT = (257, 300, 320, 321, 384, 385, 513, 576, 640, 641, 1025, 1345, 256, 512)
ALONE = (1, 60, 64, 65, 100, 128, 129, 200, 255, 0)
CASES = {
    # rows of the experts, H, F (column tiles: F / 128 in layer0, H / 256 in layer1), beside in layer0 / layer1 with 256-row tiles
    "few_tiles_behind": (FULL_AND_LIGHT + ALONE, 256, 128, False, False),
    "few_tiles_beside": (FULL_AND_LIGHT + ALONE, 256, 2304, True, False),
    "many_tiles_layer0_only": (FULL_AND_LIGHT * 4 + ALONE * 3, 256, 512, True, False),
    "many_tiles_both": ((290,) * 48 + ALONE, 1024, 384, True, True),
    "many_tiles_behind": ((2100,) * 10 + (257, 1) * 10, 256, 384, False, False),
}


def _beside(rows, tile_m, block_m, n_tiles_n):
    """Whether the light tiles of a layer lie in the blocks of the full ones."""
    import gpu_harness as H
    near = sum(tile_m < r <= (block_m + 1) * tile_m and 0 < r % tile_m and bool(H.height_class(r % tile_m) < H.height_class(tile_m)) for r in rows)
    return near * n_tiles_n >= 128


@pytest.mark.parametrize("name", CASES)
def test_remainders_beside_full_tiles(name):
    import gpu_harness as H
    import paper_2502_19811_amd as moe
    rows, Hd, F, in0, in1 = CASES[name]
    assert (_beside(rows, 256, 4, F // 128), _beside(rows, 256, 4, Hd // 256)) == (in0, in1)
    cfg = wl.MoEConfig(name, T=sum(rows), H=Hd, F=F, E=len(rows), k=1, act=wl.ACT_SWIGLU, S=4, seed=840)
    inp = wl.make_inputs(cfg, threads=4)
    ids = np.repeat(np.arange(cfg.E, dtype=np.int32), rows)[np.random.default_rng(8).permutation(cfg.T)][:, None].copy()
    w = np.linspace(0.5, 1.5, cfg.T, dtype=np.float32)[:, None].copy()
    ref = orc.moe_layer(inp.x, inp.W1, inp.W2, ids, w, cfg.act)
    counts, offsets, perm, _ = orc.build_permutation(ids, cfg.E)
    first = None
    for tile_m in (256, 128):
        for options, kw in (({}, {}), ({"layer0_order": 2, "layer0_waves": 3}, {"waves": (3, 4)}), ({"block_m": 1}, {}),
                            ({"layer0_order": 1, "layer1_order": 1}, {}), ({"large_schedule": 1}, None)):
            print(f"light tiles {name} tile_m {tile_m} {options}", flush=True)
            layer = H.GpuLayer(cfg, inp, ids, w, {"tile_m": tile_m, **options}, packed=True)
            layer.forward()
            run = layer.results()
            assert run.status == 0
            H.check_tile_table(run.tiles, cfg, offsets, perm, inp.seg_offsets, tile_m)
            if kw is not None:
                by_segment = options.get("layer0_order") == 1
                beside = lambda n: not by_segment and _beside(rows, tile_m, options.get("block_m", 4), n)
                H.check_schedule(*layer.schedule(0), run.tiles, F // 128, seg_major=by_segment, beside=beside(F // 128), **kw)
                H.check_schedule(*layer.schedule(1), run.tiles, Hd // 256, panel_major=by_segment, beside=beside(Hd // 256))
            layer.close()
            if first is None:
                first = run.out
                a, b = H.error_metrics(first, ref)
                assert a <= H.REL_TOL and b <= H.REL_TOL, f"{a:.3e} {b:.3e}"
            np.testing.assert_array_equal(run.out, first)
