"""The GroupGEMM of small batches against the oracle, at the sizes where it changes its shape: 8 / 9 and 16 / 17 tokens
(8, 16 and 32 rows per unit), experts with more rows than a unit holds, reduction lengths that the ring of operands does not
divide, and the first batch beyond it (tile kernel)."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import moe_oracle as orc

pytestmark = pytest.mark.gpu

SIZES = [
    # T, H, F, E, k, act
    (1, 1280, 1152, 8, 2, wl.ACT_SWIGLU),
    (8, 1280, 1152, 8, 2, wl.ACT_SWIGLU),
    (9, 1280, 1152, 8, 2, wl.ACT_SWIGLU),
    (16, 1024, 1280, 8, 2, wl.ACT_GELU),
    (17, 2304, 1280, 8, 2, wl.ACT_GELU),
    (64, 1280, 1152, 8, 2, wl.ACT_SWIGLU),
    (65, 1280, 1152, 8, 2, wl.ACT_SWIGLU),
    (3, 2048, 2176, 64, 16, wl.ACT_SWIGLU),
]


@pytest.mark.parametrize("size", SIZES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("packed", [False, True], ids=["plain", "packed"])
def test_small_batches_match_the_oracle(size, packed):
    import gpu_harness as H
    T, Hd, F, E, k, act = size
    cfg = wl.MoEConfig("decode", T=T, H=Hd, F=F, E=E, k=k, act=act, S=3, seed=600 + T)
    inp = wl.make_inputs(cfg, threads=4)
    routed, w = orc.route_topk(inp.logits, k)
    crowded = np.tile(np.arange(E - k, E, dtype=np.int32), (T, 1))     # every token to the same k experts: T rows each
    for ids in (routed, crowded):
        print(f"decode {size} packed {packed} rows of the fullest expert {np.bincount(ids.ravel()).max()}", flush=True)
        ref = orc.moe_layer(inp.x, inp.W1, inp.W2, ids, w, act)
        layer = H.GpuLayer(cfg, inp, ids, w, packed=packed)
        # nothing is written behind the output or the workspace (Y, layer1's output, is the last part of it)
        n = layer.ws.numel()
        ws = torch.full((n + (1 << 20),), 0x5A, dtype=torch.uint8, device="cuda")
        out = torch.full((T + 64, Hd), 7.0, dtype=torch.bfloat16, device="cuda")
        layer.ws, layer.out = ws[:n], out[:T]
        layer.forward(); run = layer.results()
        assert run.status == 0
        assert bool((ws[n:] == 0x5A).all()) and bool((out[T:] == 7.0).all())
        a, b = H.error_metrics(run.out, ref)
        print(f"  err {a:.3e} {b:.3e}", flush=True)
        assert a <= H.REL_TOL and b <= H.REL_TOL
        # ready flags that are all there
        layer.out.fill_(7.0)
        layer.forward(seg_ready=torch.ones(cfg.S, dtype=torch.int32, device="cuda"), epoch=1)
        np.testing.assert_array_equal(layer.results().out, run.out)
        layer.close()


def test_small_batch_with_a_missing_flag_times_out():
    import gpu_harness as H
    cfg = wl.MoEConfig("decode_flag", T=12, H=1280, F=1152, E=4, k=2, act=wl.ACT_SWIGLU, S=2, seed=650)
    inp = wl.make_inputs(cfg, threads=4)
    ids, w = orc.route_topk(inp.logits, cfg.k)
    layer = H.GpuLayer(cfg, inp, ids, w, {"spin_limit": 200}, packed=True)
    flags = torch.tensor([1, 0], dtype=torch.int32, device="cuda")
    print("decode with a flag that never arrives", flush=True)
    layer.forward(seg_ready=flags, epoch=1)
    assert layer.results().status == -6
    flags[1] = 1
    layer.forward(seg_ready=flags, epoch=1)
    run = layer.results()
    layer.close()
    assert run.status == 0
    a, b = H.error_metrics(run.out, orc.moe_layer(inp.x, inp.W1, inp.W2, ids, w, cfg.act))
    assert a <= H.REL_TOL and b <= H.REL_TOL


@pytest.mark.parametrize("fill", [0, 0xFF])
@pytest.mark.parametrize("Hd,F", [(256, 2048), (4096, 128)], ids=["layer1_alone", "layer0_alone"])
def test_one_layer_alone_in_small_batches(Hd, F, fill):
    """Plain weights of 256 experts: one GroupGEMM has fewer tiles than the device has compute units and the other more, and
    both schedules together are more items than the one-workgroup index build takes.  Nothing may depend on what the
    workspace held before."""
    import gpu_harness as H
    cfg = wl.MoEConfig("decode_mixed", T=2, H=Hd, F=F, E=256, k=8, act=wl.ACT_SWIGLU, S=1, seed=660)
    inp = wl.make_inputs(cfg, threads=2, weights=False)
    ids, w = orc.route_topk(inp.logits, cfg.k)
    used = np.unique(ids)
    inp.W1 = np.zeros((cfg.E, Hd, 2 * F), np.uint16)
    inp.W2 = np.zeros((cfg.E, F, Hd), np.uint16)
    inp.W1[used] = wl.normal_bf16((used.size, Hd, 2 * F), 661, 1, Hd ** -0.5)
    inp.W2[used] = wl.normal_bf16((used.size, F, Hd), 661, 2, F ** -0.5)
    ref = orc.moe_layer(inp.x, inp.W1, inp.W2, ids, w, cfg.act)
    layer = H.GpuLayer(cfg, inp, ids, w)
    layer.ws.fill_(fill)
    print(f"decode mixed H {Hd} F {F} workspace filled with {fill}", flush=True)
    layer.forward()
    run = layer.results()
    layer.close()
    assert run.status == 0
    a, b = H.error_metrics(run.out, ref)
    assert a <= H.REL_TOL and b <= H.REL_TOL, f"{a:.3e} {b:.3e}"


def test_an_expert_of_more_than_4_gib():
    """Two tokens of one expert whose W1 is 16 GiB: beyond what 32-bit byte offsets inside an expert reach.  Checked against a plain
    product in fp32 of the same tensors."""
    import gpu_harness as H
    import paper_2502_19811_amd as moe
    T, Hd, F = 2, 131840, 32640
    g = torch.Generator(device="cuda")
    g.manual_seed(680)

    def normal(shape, std):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)

    x, W1, W2 = normal((T, Hd), 1.0), normal((1, Hd, 2 * F), Hd ** -0.5), normal((1, F, Hd), F ** -0.5)
    a = torch.zeros((T, 2 * F), device="cuda")
    for k in range(0, Hd, 8240):
        a += x[:, k:k + 8240].float() @ W1[0, k:k + 8240].float()
    h = (torch.nn.functional.silu(a[:, :F]) * a[:, F:]).to(torch.bfloat16)
    ref = torch.zeros((T, Hd), device="cuda")
    for k in range(0, F, 4080):
        ref += h[:, k:k + 4080].float() @ W2[0, k:k + 4080].float()
    plan = moe.moe_plan_create(T, Hd, F, 1, 1, 1, moe.MOE_ACT_SWIGLU, [0, T])
    ws = torch.zeros(moe.moe_plan_workspace_bytes(plan), dtype=torch.uint8, device="cuda")
    ids, w = torch.zeros((T, 1), dtype=torch.int32, device="cuda"), torch.ones((T, 1), device="cuda")
    out = torch.zeros((T, Hd), dtype=torch.bfloat16, device="cuda")
    print("decode, expert of 16 GiB", flush=True)
    moe.moe_layer_forward(plan, x, ids, w, W1, W2, moe.MOE_ACT_SWIGLU, out, ws)
    assert moe.moe_last_device_status(plan, ws) == 0
    moe.moe_plan_destroy(plan)
    a, b = H.error_metrics(H.bf16_to_np(out), ref.double().cpu().numpy())
    assert a <= H.REL_TOL and b <= H.REL_TOL, f"{a:.3e} {b:.3e}"


def _bits(layer):
    layer.forward()
    run = layer.results()
    assert run.status == 0
    return layer.out.view(torch.int16).cpu().numpy().copy(), run


@pytest.mark.parametrize("T,act", [(1, wl.ACT_SWIGLU), (7, wl.ACT_SWIGLU), (12, wl.ACT_GELU), (33, wl.ACT_SWIGLU)])
def test_a_small_batch_has_the_bits_of_every_other_way_to_compute_it(T, act):
    """Reductions longer than 1024: packed and plain weights, the options that bypass the kernel of small batches, and a larger
    batch around the same tokens all sum in the same order."""
    import gpu_harness as H
    cfg = wl.MoEConfig("decode_bits", T=T, H=2304, F=1792, E=8, k=2, act=act, S=1, seed=670)
    big = wl.scaled(cfg, T=300)
    inp_big = wl.make_inputs(big, threads=4)
    ids_big, w_big = orc.route_topk(inp_big.logits, cfg.k)
    ids, w = ids_big[:T].copy(), w_big[:T].copy()
    inp = wl.MoEInputs(cfg, inp_big.x[:T].copy(), inp_big.W1, inp_big.W2, inp_big.logits[:T], np.array([0, T], np.int32))
    layer = H.GpuLayer(big, inp_big, ids_big, w_big)
    want = _bits(layer)[0][:T]
    layer.close()
    for packed in (False, True):
        for opts in ({}, {"n_cu": 256}, {"layer1_order": 1}, {"fuse_layers": 1}, {"large_schedule": 1}, {"handoff_fences": 1}):
            print(f"decode bits T {T} act {act} packed {packed} {opts}", flush=True)
            layer = H.GpuLayer(cfg, inp, ids, w, opts, packed=packed)
            got, run = _bits(layer)
            layer.close()
            np.testing.assert_array_equal(got, want)
    a, b = H.error_metrics(run.out, orc.moe_layer(inp.x, inp.W1, inp.W2, ids, w, act))
    assert a <= H.REL_TOL and b <= H.REL_TOL


@pytest.mark.parametrize("T,E,k,act,tile_m,Hd,F", [(256, 256, 16, wl.ACT_SWIGLU, 64, 256, 128), (128, 256, 16, wl.ACT_SWIGLU, 64, 512, 512),
                                                   (256, 128, 8, wl.ACT_GELU, 256, 512, 512), (40, 20, 8, wl.ACT_SWIGLU, 128, 512, 512)])
def test_every_row_part_of_crowded_experts(T, E, k, act, tile_m, Hd, F):
    """One expert with every token, others with a few or none: several row parts of one expert beside single ones of others, more
    tiles than a wavefront has lanes.  The tile kernel (option n_cu) gives the same bits."""
    import gpu_harness as H
    cfg = wl.MoEConfig("decode_parts", T=T, H=Hd, F=F, E=E, k=k, act=act, S=1, seed=690)
    inp = wl.make_inputs(cfg, threads=4)
    rng = np.random.default_rng(690)
    ids = np.stack([np.concatenate([[E // 3], rng.permutation(np.delete(np.arange(E), E // 3))[:k - 1]]) for _ in range(T)]).astype(np.int32)
    w = rng.uniform(0.1, 1.0, (T, k)).astype(np.float32)
    for packed in (False, True):
        print(f"decode parts T {T} E {E} k {k} act {act} tile_m {tile_m} packed {packed}", flush=True)
        bits = []
        for opts in ({"tile_m": tile_m}, {"tile_m": tile_m, "n_cu": 256}):
            layer = H.GpuLayer(cfg, inp, ids, w, opts, packed=packed)
            got, run = _bits(layer)
            layer.close()
            bits.append(got)
        np.testing.assert_array_equal(bits[0], bits[1])
    a, b = H.error_metrics(run.out, orc.moe_layer(inp.x, inp.W1, inp.W2, ids, w, act))
    assert a <= H.REL_TOL and b <= H.REL_TOL


@pytest.mark.parametrize("packed", [False, True], ids=["plain", "packed"])
def test_a_missing_segment_costs_its_own_rows_only(packed):
    """Tokens of the first segment use the first experts, tokens of the second one the others; the second never arrives."""
    import gpu_harness as H
    cfg = wl.MoEConfig("decode_half", T=20, H=512, F=1152, E=8, k=2, act=wl.ACT_SWIGLU, S=2, seed=651)
    inp = wl.make_inputs(cfg, threads=4)
    half = int(inp.seg_offsets[1])
    rng = np.random.default_rng(651)
    ids = np.stack([rng.permutation(4)[:2] + (0 if t < half else 4) for t in range(cfg.T)]).astype(np.int32)
    w = rng.uniform(0.1, 1.0, (cfg.T, 2)).astype(np.float32)
    layer = H.GpuLayer(cfg, inp, ids, w, {"spin_limit": 200}, packed=packed)
    layer.forward()
    want = layer.results().out
    layer.out.fill_(7.0)
    print(f"decode, second of two segments missing, packed {packed}", flush=True)
    layer.ws.zero_()
    layer.forward(seg_ready=torch.tensor([3, 2], dtype=torch.int32, device="cuda"), epoch=3)
    run = layer.results()
    layer.close()
    assert run.status == -6
    np.testing.assert_array_equal(run.out[:half], want[:half])


@pytest.mark.parametrize("packed", [False, True], ids=["plain", "packed"])
def test_segments_that_arrive_during_the_forward(packed):
    """The receive buffer is filled segment by segment while a small batch waits for it.  The wait is bounded, so that a lost segment
    fails the test."""
    import gpu_harness as H
    import paper_2502_19811_amd as moe
    cfg = wl.MoEConfig("decode_arrival", T=33, H=1024, F=1792, E=8, k=2, act=wl.ACT_SWIGLU, S=4, seed=652)
    inp = wl.make_inputs(cfg, threads=4)
    ids, w = orc.route_topk(inp.logits, cfg.k)
    layer = H.GpuLayer(cfg, inp, ids, w, {"spin_limit": 1 << 21}, packed=packed)
    want, _ = _bits(layer)
    staging = layer.x.clone()
    layer.x.zero_()
    layer.out.zero_()
    flags = torch.zeros(cfg.S, dtype=torch.int32, device="cuda")
    counters = torch.zeros(cfg.S, dtype=torch.int32, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    print(f"decode with arriving segments, packed {packed}", flush=True)
    moe.moe_play_arrival(layer.plan, staging, layer.x, flags, counters, 3, 0.2, 2, side)   # 67 KB at 0.2 GB/s: 0.3 ms
    layer.forward(seg_ready=flags, epoch=3)
    torch.cuda.synchronize()
    run = layer.results()
    got = layer.out.view(torch.int16).cpu().numpy()
    layer.close()
    assert run.status == 0
    np.testing.assert_array_equal(got, want)


def test_schedules_a_small_batch_did_without_belong_to_the_workspace():
    """One plan, two workspaces: the first has seen a forward that needs no tile schedules, the second one that builds them.  The
    steps after the index build, and the schedule itself, are then asked of the first with the option of the second, and the reverse."""
    import gpu_harness as H
    import paper_2502_19811_amd as moe
    cfg = wl.MoEConfig("decode_two_ws", T=24, H=512, F=1152, E=8, k=2, act=wl.ACT_SWIGLU, S=2, seed=653)
    inp = wl.make_inputs(cfg, threads=4)
    ids, w = orc.route_topk(inp.logits, cfg.k)
    layer = H.GpuLayer(cfg, inp, ids, w, packed=True)
    want, run = _bits(layer)
    first, second = layer.ws, torch.zeros_like(layer.ws)
    moe.moe_plan_set_option(layer.plan, "handoff_fences", 1)      # the tile kernel
    layer.ws = second
    layer.forward()
    for ws, fences in ((first, 1), (second, 0), (first, 0), (second, 1)):
        print(f"phases without the index build, {'first' if ws is first else 'second'} workspace, fences {fences}", flush=True)
        moe.moe_plan_set_option(layer.plan, "handoff_fences", fences)
        moe.moe_plan_set_option(layer.plan, "phases", 14)
        layer.ws = ws
        layer.out.fill_(7.0)
        got, _ = _bits(layer)
        np.testing.assert_array_equal(got, want)
        for l, n in ((0, cfg.F // 128), (1, cfg.H // 256)):
            items, queues = layer.schedule(l)
            H.check_schedule(items, queues, run.tiles, n)
    layer.close()
