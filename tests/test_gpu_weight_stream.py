"""Weight loads with and without the non-temporal hint: batches on both sides of the two rules that choose between them (the
weights a forward reads against half the Infinity Cache, the rows per expert), in every kernel that has them.  A token's output
has the same bits in all of them, and is that of a plain computation in fp32."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# tokens: 1 reads two experts of 31 MB, 3 and more read over 128 MB; 1280 are 320 rows per expert, 1281 more
SIZES = (1, 3, 16, 40, 200, 1280, 1281)


@pytest.mark.parametrize("packed", [False, True], ids=["plain", "packed"])
@pytest.mark.parametrize("act", ["swiglu", "gelu"])
def test_outputs_do_not_depend_on_how_weights_are_loaded(act, packed):
    import gpu_harness as G
    import paper_2502_19811_amd as moe
    E, k, H, F = 8, 2, 2048, 2560 if act == "swiglu" else 3840
    F1, kind = (2 * F, moe.MOE_ACT_SWIGLU) if act == "swiglu" else (F, moe.MOE_ACT_GELU)
    T = SIZES[-1]
    g = torch.Generator(device="cuda")
    g.manual_seed(90)
    bf16 = lambda shape, std: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)
    x, W1, W2 = bf16((T, H), 1.0), bf16((E, H, F1), H ** -0.5), bf16((E, F, H), F ** -0.5)
    w, ids = torch.softmax(torch.empty((T, E), device="cuda").normal_(generator=g), 1).topk(k)
    ids, w = ids.to(torch.int32).contiguous(), (w / w.sum(1, keepdim=True)).contiguous()
    ref = torch.zeros((T, H), device="cuda")
    for e in range(E):
        t, j = (ids == e).nonzero(as_tuple=True)
        a = x[t].float() @ W1[e].float()
        h = torch.nn.functional.silu(a[:, :F]) * a[:, F:] if act == "swiglu" else torch.nn.functional.gelu(a)
        ref.index_add_(0, t, (h.bfloat16().float() @ W2[e].float()) * w[t, j][:, None])
    ref = ref.double().cpu().numpy()

    outs = {}
    for n in SIZES:
        print(f"weight stream {act} packed {packed} tokens {n}", flush=True)
        plan = moe.moe_plan_create(n, H, F, E, k, 1, kind, [0, n])
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
        outs[n] = G.bf16_to_np(out)
        a, b = G.error_metrics(outs[n], ref[:n])
        assert a <= G.REL_TOL and b <= G.REL_TOL, f"{n} tokens: {a:.3e} {b:.3e}"
    for n in SIZES[:-1]:
        np.testing.assert_array_equal(outs[n], outs[T][:n])
