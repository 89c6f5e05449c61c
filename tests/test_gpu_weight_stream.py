"""Weight loads with and without the non-temporal hint: batches on both sides of the rules that choose between them (the
weights a forward reads against half the Infinity Cache, the rows per expert on average, the rows of an expert against the
height of the tiles), in every kernel and tile variant that has them.  A token's output
has the same bits in all of them, and is that of a plain computation in fp32."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# tokens: 1 reads two experts of 31 MB, 3 and more read over 128 MB; 976 are 244 rows per expert, 977 more
SIZES = (1, 3, 16, 40, 200, 976, 977, 1280, 1281)
# Popularity falling as rank^-0.9: experts of one tile (weights loaded with the hint) and of several (without it) in one launch, in tiles of
# all four heights; the first is beyond the rows per expert of the rule and has none with it
TILED = [(1281, 0), (300, 64), (300, 128), (560, 64), (560, 128), (560, 256), (900, 128), (900, 256)]   # (tokens, tile_m)


def outputs(act, packed, seed, runs, crowding):
    """Outputs of the first n tokens of one batch, for each (n, tile_m) of runs (tile_m 0: the plan's choice), each checked
    against the fp32 computation; popularity of expert e falls as (e + 1)^-crowding."""
    import gpu_harness as G
    import paper_2502_19811_amd as moe
    E, k, H, F = 8, 2, 2048, 2560 if act == "swiglu" else 3840
    F1, kind = (2 * F, moe.MOE_ACT_SWIGLU) if act == "swiglu" else (F, moe.MOE_ACT_GELU)
    T = max(n for n, _ in runs)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    bf16 = lambda shape, std: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)
    x, W1, W2 = bf16((T, H), 1.0), bf16((E, H, F1), H ** -0.5), bf16((E, F, H), F ** -0.5)
    logits = torch.empty((T, E), device="cuda").normal_(generator=g) - crowding * torch.log(torch.arange(1, E + 1, device="cuda"))
    w, ids = torch.softmax(logits, 1).topk(k)
    ids, w = ids.to(torch.int32).contiguous(), (w / w.sum(1, keepdim=True)).contiguous()
    ref = torch.zeros((T, H), device="cuda")
    for e in range(E):
        t, j = (ids == e).nonzero(as_tuple=True)
        a = x[t].float() @ W1[e].float()
        h = torch.nn.functional.silu(a[:, :F]) * a[:, F:] if act == "swiglu" else torch.nn.functional.gelu(a)
        ref.index_add_(0, t, (h.bfloat16().float() @ W2[e].float()) * w[t, j][:, None])
    ref = ref.double().cpu().numpy()

    outs = {}
    for n, tile_m in runs:
        counts = torch.bincount(ids[:n].flatten(), minlength=E).tolist()
        print(f"weight stream {act} packed {packed} tokens {n} tile_m {tile_m} rows {counts}", flush=True)
        plan = moe.moe_plan_create(n, H, F, E, k, 1, kind, [0, n])
        if tile_m:
            moe.moe_plan_set_option(plan, "tile_m", tile_m)
        B1, B2 = W1, W2
        if packed:
            B1, B2 = torch.empty_like(W1), torch.empty_like(W2)
            moe.moe_pack_weights(plan, W1, W2, B1, B2)
            moe.moe_plan_set_option(plan, "weights_packed", 1)
        ws = torch.zeros(moe.moe_plan_workspace_bytes(plan), dtype=torch.uint8, device="cuda")
        out = torch.full((n, H), 7.0, dtype=torch.bfloat16, device="cuda")
        moe.moe_layer_forward(plan, x[:n], ids[:n], w[:n], B1, B2, kind, out, ws)
        assert moe.moe_last_device_status(plan, ws) == 0
        moe.moe_plan_destroy(plan)
        outs[n, tile_m] = G.bf16_to_np(out)
        a, b = G.error_metrics(outs[n, tile_m], ref[:n])
        assert a <= G.REL_TOL and b <= G.REL_TOL, f"{n} tokens: {a:.3e} {b:.3e}"
        # experts of one tile and of several, in the same launch
        if tile_m:
            assert min(c for c in counts if c) <= tile_m < max(counts)
    return outs


@pytest.mark.parametrize("packed", [False, True], ids=["plain", "packed"])
@pytest.mark.parametrize("act", ["swiglu", "gelu"])
def test_outputs_do_not_depend_on_how_weights_are_loaded(act, packed):
    outs = outputs(act, packed, 90, [(n, 0) for n in SIZES], 0.0)
    for n in SIZES[:-1]:
        np.testing.assert_array_equal(outs[n, 0], outs[SIZES[-1], 0][:n])


@pytest.mark.parametrize("packed", [False, True], ids=["plain", "packed"])
@pytest.mark.parametrize("act", ["swiglu", "gelu"])
def test_outputs_do_not_depend_on_whose_weights_are_streamed(act, packed):
    outs = outputs(act, packed, 91, TILED, 0.9)
    for n, tile_m in TILED[1:]:
        np.testing.assert_array_equal(outs[n, tile_m], outs[TILED[0]][:n])
