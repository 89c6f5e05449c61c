"""A plan that fits the library's own 32 MiB workspace with 256-row tiles fits it with the tile height the plan chooses."""
import paper_2502_19811_amd as moe

LIMIT = 32 << 20


def test_the_chosen_tile_height_does_not_outgrow_the_static_workspace():
    shorter_would_not_fit = 0
    for T in range(30000, 33000, 10):
        plan = moe.moe_plan_create(T, 256, 256, 4, 1, 1, moe.MOE_ACT_GELU, [0, T])
        chosen = moe.moe_plan_workspace_bytes(plan)
        by_height = {}
        for tile_m in (128, 256):
            moe.moe_plan_set_option(plan, "tile_m", tile_m)
            by_height[tile_m] = moe.moe_plan_workspace_bytes(plan)
        moe.moe_plan_destroy(plan)
        assert chosen <= LIMIT or by_height[256] > LIMIT
        shorter_would_not_fit += by_height[128] > LIMIT >= by_height[256]
    assert shorter_would_not_fit > 0
