"""The one-workgroup index build at the edges of its range: a batch of one pair, one beyond a wavefront's run of 64 pairs,
the last one it takes and the first that goes to the three kernels; all experts, one expert, ids out of range."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import moe_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,k", [(1, 1, 1), (1, 256, 16), (65, 3, 1), (600, 64, 3), (4096, 5, 1), (2048, 8, 2), (256, 256, 16),
                                   (2049, 8, 2)])
@pytest.mark.parametrize("tile_m", [64, 256])
def test_index_outputs_and_schedules_of_small_batches(T, E, k, tile_m):
    import gpu_harness as H
    cfg = wl.MoEConfig("small_index", T=T, H=512, F=512, E=E, k=k, act=wl.ACT_SWIGLU, S=5, seed=700)
    print(f"index T {T} E {E} k {k} tile_m {tile_m}", flush=True)
    inp = wl.make_inputs(cfg, threads=2, weights=False)
    routed, w = orc.route_topk(inp.logits, k)
    same = np.tile(np.arange(E - k, E, dtype=np.int32), (T, 1))
    for ids in (routed, same):
        layer = H.GpuLayer(cfg, inp, ids, w, {"phases": 1, "tile_m": tile_m})
        layer.forward()
        run = layer.results()
        counts, offsets, perm, inv = orc.build_permutation(ids, E)
        np.testing.assert_array_equal(run.counts, counts)
        np.testing.assert_array_equal(run.offsets, offsets)
        np.testing.assert_array_equal(run.perm, perm)
        np.testing.assert_array_equal(run.inv_perm, inv)
        H.check_tile_table(run.tiles, cfg, offsets, perm, inp.seg_offsets, tile_m)
        for l, n in ((0, cfg.F // 128), (1, cfg.H // 256)):     # (also when the forward itself had no use for them)
            items, queues = layer.schedule(l)
            H.check_schedule(items, queues, run.tiles, n)
        assert run.status == 0
        bad = ids.copy()
        bad[T // 2, 0] = E
        layer.ids.copy_(torch.from_numpy(bad).cuda())
        layer.forward()
        assert layer.results().status == -1
        layer.close()


@pytest.mark.parametrize("T", [600, 3000])
def test_the_schedule_of_a_flagged_forward_follows_what_has_arrived(T):
    """All segments there when the schedule is built: the order of resident input.  One missing: waves of segments."""
    import gpu_harness as H
    import paper_2502_19811_amd as moe
    cfg = wl.MoEConfig("arrived", T=T, H=512, F=2560, E=8, k=2, act=wl.ACT_SWIGLU, S=8, seed=701)
    inp = wl.make_inputs(cfg, threads=2, weights=False)
    ids, w = orc.route_topk(inp.logits, cfg.k)
    layer = H.GpuLayer(cfg, inp, ids, w, {"phases": 1, "block_m": 2, "tile_m": 64})
    n_waves = moe.moe_plan_get_option(layer.plan, "layer0_waves")
    layer.forward()
    resident, queues = layer.schedule(0)
    flags = torch.full((cfg.S,), 4, dtype=torch.int32, device="cuda")
    layer.forward(seg_ready=flags, epoch=4)
    there, there_queues = layer.schedule(0)
    assert there_queues == queues
    for first, count, stride in queues:
        np.testing.assert_array_equal(there[first:first + count * stride:stride], resident[first:first + count * stride:stride])
    flags[5] = 3
    layer.forward(seg_ready=flags, epoch=4)
    items, queues = layer.schedule(0)
    H.check_schedule(items, queues, layer.results().tiles, cfg.F // 128, waves=(n_waves, cfg.S))
    layer.close()
