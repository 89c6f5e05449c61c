"""Queues of tiles: whatever the order of a schedule, where its queue heads lie and how many workgroups walk it (queues of
less than a round, of a few rounds and of many), every tile is computed once.  The plan's options change from forward to
forward on one workspace, and the schedules of a forward are run again; all outputs have the same bits."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import moe_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hd,F,act", [(256, 512, wl.ACT_GELU), (1536, 640, wl.ACT_SWIGLU)], ids=["little_room", "spread"])
def test_every_order_and_workgroup_count_gives_the_same_bits(Hd, F, act):
    import gpu_harness as H
    import paper_2502_19811_amd as moe
    cfg = wl.MoEConfig("queues", T=1111, H=Hd, F=F, E=6, k=2, act=act, S=4, seed=820)
    inp = wl.make_inputs(cfg, threads=4)
    ids, w = orc.route_topk(inp.logits, cfg.k)
    ref = orc.moe_layer(inp.x, inp.W1, inp.W2, ids, w, act)
    layer = H.GpuLayer(cfg, inp, ids, w)
    first = None
    for n_cu in (256, 8, 40, 64):
        moe.moe_plan_set_option(layer.plan, "n_cu", n_cu)
        for order0, order1 in ((0, 0), (1, 1), (2, 0), (1, 0), (0, 2), (0, 1)):
            moe.moe_plan_set_option(layer.plan, "layer0_order", order0)
            moe.moe_plan_set_option(layer.plan, "layer1_order", order1)
            for phases in (15, 14):      # with the index build, then its schedules again
                print(f"queues H {Hd} n_cu {n_cu} orders {order0} {order1} phases {phases}", flush=True)
                moe.moe_plan_set_option(layer.plan, "phases", phases)
                layer.out.fill_(7.0)
                layer.forward()
                run = layer.results()
                assert run.status == 0
                if first is None:
                    first = run.out
                    a, b = H.error_metrics(first, ref)
                    assert a <= H.REL_TOL and b <= H.REL_TOL
                np.testing.assert_array_equal(run.out, first)
            # the layer1 order changes between the index build and the forward that runs its schedules again
            if order1 == 1:
                moe.moe_plan_set_option(layer.plan, "layer1_order", 0)
                layer.out.fill_(7.0)
                layer.forward()
                np.testing.assert_array_equal(layer.results().out, first)
            moe.moe_plan_set_option(layer.plan, "phases", 15)
    layer.close()


@pytest.mark.parametrize("T,Hd,F", [(16, 256, 4096), (64, 256, 2048), (64, 768, 2048), (64, 1280, 2048)])
def test_heads_of_a_schedule_made_later(T, Hd, F):
    """A small batch leaves its schedules out; the steps after the index build, asked for with another kind of schedule, make them up in
    the workspace, and a second workspace that has seen the usual kind comes in between.  Nothing is written behind the workspace
    (Y and the queue heads are the last of it)."""
    import gpu_harness as H
    import paper_2502_19811_amd as moe
    cfg = wl.MoEConfig("heads_later", T=T, H=Hd, F=F, E=8, k=2, act=wl.ACT_SWIGLU, S=2, seed=830)
    inp = wl.make_inputs(cfg, threads=4)
    ids, w = orc.route_topk(inp.logits, cfg.k)
    layer = H.GpuLayer(cfg, inp, ids, w, packed=True)
    n, guard = layer.ws.numel(), 1 << 20
    spaces = [torch.full((n + guard,), 0x5A, dtype=torch.uint8, device="cuda") for _ in range(2)]
    want = None

    def forward(space, phases, **options):
        nonlocal want
        for name in ("layer1_order", "large_schedule"):
            moe.moe_plan_set_option(layer.plan, name, options.get(name, 0))
        moe.moe_plan_set_option(layer.plan, "phases", phases)
        print(f"heads T {T} H {Hd} F {F} workspace {space} phases {phases} {options}", flush=True)
        layer.ws = spaces[space][:n]
        layer.out.fill_(7.0)
        layer.forward()
        run = layer.results()
        assert run.status == 0
        if want is None:
            want = run.out
            a, b = H.error_metrics(want, orc.moe_layer(inp.x, inp.W1, inp.W2, ids, w, cfg.act))
            assert a <= H.REL_TOL and b <= H.REL_TOL
        np.testing.assert_array_equal(run.out, want)
        assert bool((spaces[space][n:] == 0x5A).all())

    for options in ({"layer1_order": 1}, {"large_schedule": 1}):
        forward(0, 15)                  # index build without schedules
        forward(0, 14, **options)       # ... made up
        forward(0, 14, **options)       # ... run again
    forward(0, 15, layer1_order=1)
    forward(1, 15)
    forward(0, 14, layer1_order=1)      # the first workspace's schedule, after the usual kind on the second
    forward(1, 14)
    layer.close()
