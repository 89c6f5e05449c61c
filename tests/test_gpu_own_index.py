"""Small batches whose GroupGEMMs make their index themselves: pair counts at the edges of the runs of 64 they are ranked in and
of the limit, from which on a launch of its own makes the index; few and many experts, none with rows for most of them, all
rows on one; ready flags; ids that are no expert.  Index, tile table and schedules in the workspace are those of every other
forward.  And the largest batches of weights that fit in an L2."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import moe_oracle as orc

pytestmark = pytest.mark.gpu

CASES = [
    # T, H, F, E, k, act
    (1, 256, 256, 4, 1, wl.ACT_GELU),
    (63, 256, 128, 8, 1, wl.ACT_SWIGLU),
    (65, 512, 256, 5, 1, wl.ACT_SWIGLU),
    (32, 256, 128, 128, 8, wl.ACT_SWIGLU),      # 256 pairs, the last batch of so many experts with an index of its own
    (65, 256, 128, 128, 4, wl.ACT_SWIGLU),
    (32, 256, 128, 256, 16, wl.ACT_SWIGLU),
    (128, 256, 128, 64, 3, wl.ACT_SWIGLU),      # 384 pairs, the last batch
    (385, 256, 128, 25, 1, wl.ACT_SWIGLU),
    (171, 256, 128, 64, 3, wl.ACT_SWIGLU),
    (192, 256, 512, 4, 2, wl.ACT_GELU),         # 384 pairs, 96 rows per expert
    (256, 256, 512, 4, 2, wl.ACT_GELU),         # 512 pairs, 128 rows per expert
    (257, 256, 512, 4, 2, wl.ACT_GELU),
    (2048, 256, 512, 4, 2, wl.ACT_GELU),        # 4096 pairs, the last such batch; 1366 of 3 experts
    (2049, 256, 512, 4, 2, wl.ACT_GELU),
    (1365, 256, 384, 3, 3, wl.ACT_SWIGLU),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_index_and_outputs(case):
    import gpu_harness as H
    import paper_2502_19811_amd as moe
    T, Hd, F, E, k, act = case
    cfg = wl.MoEConfig("own_index", T=T, H=Hd, F=F, E=E, k=k, act=act, S=5, seed=860 + T)
    inp = wl.make_inputs(cfg, threads=4)
    routed, w = orc.route_topk(inp.logits, k)
    crowded = np.tile(np.arange(E - k, E, dtype=np.int32), (T, 1))
    n0 = F // (128 if act == wl.ACT_SWIGLU else 256)
    for packed, ids in ((True, routed), (False, routed), (False, crowded)):
        counts, offsets, perm, inv_perm = orc.build_permutation(ids, E)
        ref = orc.moe_layer(inp.x, inp.W1, inp.W2, ids, w, act)
        layer = H.GpuLayer(cfg, inp, ids, w, packed=packed)
        flags = torch.ones(cfg.S, dtype=torch.int32, device="cuda")
        for kw in ({}, {"seg_ready": flags, "epoch": 1}):
            print(f"own index {case} packed {packed} flags {bool(kw)}", flush=True)
            layer.ws.fill_(0x5A)          # nothing may depend on what the workspace held
            layer.out.fill_(7.0)
            layer.forward(**kw)
            run = layer.results()
            assert run.status == 0
            np.testing.assert_array_equal(run.counts, counts)
            np.testing.assert_array_equal(run.offsets, offsets)
            np.testing.assert_array_equal(run.perm, perm)
            np.testing.assert_array_equal(run.inv_perm, inv_perm)
            H.check_tile_table(run.tiles, cfg, offsets, perm, inp.seg_offsets, moe.moe_plan_get_option(layer.plan, "tile_m"))
            H.check_schedule(*layer.schedule(0), run.tiles, n0)
            H.check_schedule(*layer.schedule(1), run.tiles, Hd // 256)
            a, b = H.error_metrics(run.out, ref)
            assert a <= H.REL_TOL and b <= H.REL_TOL, f"{a:.3e} {b:.3e}"
        layer.close()


def test_ids_out_of_range_and_time_outs_are_reported_once():
    import gpu_harness as H
    cfg = wl.MoEConfig("own_index_status", T=20, H=256, F=256, E=6, k=2, act=wl.ACT_SWIGLU, S=2, seed=870)
    inp = wl.make_inputs(cfg, threads=2)
    ids, w = orc.route_topk(inp.logits, cfg.k)
    wrong = ids.copy()
    wrong[3, 1], wrong[17, 0] = 6, -2
    layer = H.GpuLayer(cfg, inp, wrong, w, {"spin_limit": 200})
    up, missing = (torch.tensor(f, dtype=torch.int32, device="cuda") for f in ([1, 1], [1, 0]))
    print("own index, ids that are no expert", flush=True)
    layer.forward()
    counts = np.bincount(np.where((wrong < 0) | (wrong >= 6), 5, wrong).ravel(), minlength=6)
    run = layer.results()
    assert run.status == -1
    np.testing.assert_array_equal(run.counts, counts)
    layer.ids = torch.from_numpy(ids).cuda()
    layer.forward(seg_ready=up, epoch=1)
    assert layer.results().status == 0
    layer.forward(seg_ready=missing, epoch=1)
    assert layer.results().status == -6
    layer.forward(seg_ready=up, epoch=1)
    run = layer.results()
    layer.close()
    assert run.status == 0
    a, b = H.error_metrics(run.out, orc.moe_layer(inp.x, inp.W1, inp.W2, ids, w, cfg.act))
    assert a <= H.REL_TOL and b <= H.REL_TOL


def test_time_outs_of_a_replayed_graph_belong_to_their_replay():
    """Replays of one captured forward, with and without a missing segment, and eager forwards of the plan in between: every one
    reports its own waits (the captured launches carry the serial number of the forward that was captured)."""
    import gpu_harness as H
    cfg = wl.MoEConfig("own_index_graph", T=20, H=256, F=256, E=6, k=2, act=wl.ACT_SWIGLU, S=2, seed=871)
    inp = wl.make_inputs(cfg, threads=2)
    ids, w = orc.route_topk(inp.logits, cfg.k)
    layer = H.GpuLayer(cfg, inp, ids, w, {"spin_limit": 200})
    flags = torch.ones(cfg.S, dtype=torch.int32, device="cuda")
    layer.ws.fill_(0x5A)
    layer.forward(seg_ready=flags, epoch=1)
    first = layer.results()
    assert first.status == 0
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=stream):
        layer.forward(seg_ready=flags, epoch=1, stream=stream)
    for missing in (False, True, False, True, True, False):
        print(f"own index, replay with a missing segment: {missing}", flush=True)
        flags[1] = 0 if missing else 1
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        run = layer.results()
        assert run.status == (-6 if missing else 0)
        if not missing:
            np.testing.assert_array_equal(run.out, first.out)
        flags.fill_(1)
        layer.forward(seg_ready=flags, epoch=1)
        assert layer.results().status == 0
    layer.close()
