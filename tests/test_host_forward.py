"""What the host side launches, and on which memory, followed without a GPU (host_forward.hip: the library's host code with notes in
the place of its launches)."""
import ctypes as C
import os
import subprocess

import pytest

from conftest import ROOT

INDEX, SCHEDULE, RESET, LAYER0, LAYER1, DECODE0, DECODE1 = range(1, 8)
BASE = 1 << 40          # addresses are arithmetic here, nothing is accessed
ITEM = 32               # bytes of a schedule record


class Shape(C.Structure):
    _fields_ = [(n, C.c_int32) for n in ("T", "H", "F", "E", "k", "S", "act")]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("host") / "host_forward.so")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "-O1", "-std=c++17", "-fPIC", "-shared",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2502_19811_amd", "csrc"), os.path.join(ROOT, "tests", "host_forward.hip"), "-o", so],
                   check=True, capture_output=True)
    lib = C.CDLL(so, mode=os.RTLD_LOCAL)
    lib.moe_plan_workspace_bytes.restype = C.c_size_t
    lib.moe_plan_schedule_capacity.restype = C.c_int64
    return lib


class Plan:
    def __init__(self, lib, T, H, F, E, k, act=1, S=1, **options):
        self.lib, self.act, self.p = lib, act, C.c_void_p()
        seg = (C.c_int32 * (S + 1))(*[T * s // S for s in range(S + 1)])
        assert lib.moe_plan_create(C.byref(self.p), C.byref(Shape(T, H, F, E, k, S, act)), seg) == 0
        for name, value in options.items():
            self.set(name, value)

    def set(self, name, value):
        assert self.lib.moe_plan_set_option(self.p, name.encode(), C.c_int64(value)) == 0

    def bytes(self):
        return self.lib.moe_plan_workspace_bytes(self.p)

    def forward(self, base=BASE):
        """The notes of one forward: tuples (kind, heads, stride, items0 or items, items1, own_index, stream)."""
        at = C.c_void_p(BASE >> 8)
        assert self.lib.moe_layer_forward(self.p, at, at, at, at, at, self.act, at, C.c_void_p(base), C.c_size_t(self.bytes()), None, 0, None) == 0
        out = (C.c_int64 * (7 * 32))()
        n = self.lib.host_forward_notes(out, 32)
        assert 0 < n <= 32
        return [tuple(out[7 * i:7 * i + 7]) for i in range(n)]

    def close(self):
        self.lib.moe_plan_destroy(self.p)


def check_heads(plan, notes, base=BASE):
    """Every launch of the forward has its queue heads where the launch that cleared them has, inside the workspace, and where no
    schedule can be."""
    heads = {n[1:3] for n in notes if n[0] in (INDEX, SCHEDULE, RESET, LAYER0, LAYER1) and not (n[0] == LAYER1)}
    at, stride = heads.pop()
    assert not heads
    assert all(n[1:3] == (at + 8 * stride, stride) for n in notes if n[0] == LAYER1)   # layer1's lie behind layer0's
    end = at + 15 * stride + 4
    assert base <= at and end <= base + plan.bytes()
    items = {n[3:5] for n in notes if n[0] in (INDEX, SCHEDULE, RESET)}
    assert len(items) == 1
    for layer, first in enumerate(items.pop()):
        last = first + plan.lib.moe_plan_schedule_capacity(plan.p, layer) * ITEM
        assert end <= first or at >= last, f"queue heads {at - base}..{end - base} inside the layer{layer} schedule {first - base}..{last - base}"


SHAPES = [
    # T, H, F, E, k, act
    (64, 256, 2048, 8, 2, 1), (16, 256, 4096, 8, 2, 1), (64, 768, 2048, 8, 2, 1), (64, 1280, 2048, 8, 2, 1), (24, 512, 1152, 8, 2, 1),
    (1111, 256, 512, 6, 2, 0), (1111, 1536, 640, 6, 2, 1), (8192, 4096, 14336, 8, 2, 1), (4096, 3584, 2560, 64, 8, 1), (1, 256, 256, 1, 1, 0),
    (65536, 256, 128, 256, 16, 1),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_queue_heads_lie_outside_every_schedule(lib, shape):
    """Forwards with and without the index build, the options that choose the kind of schedule changed between them, on two
    workspaces of one plan: a schedule may stem from any earlier forward."""
    for tile_m in (64, 128, 256):
        plan = Plan(lib, *shape, tile_m=tile_m, weights_packed=1)
        for order in (0, 1, 2):
            for large in (0, 1):
                for phases in (15, 14, 1, 6):
                    for base in (BASE, 2 * BASE):
                        plan.set("layer1_order", order)
                        plan.set("large_schedule", large)
                        plan.set("phases", phases)
                        notes = plan.forward(base)
                        if any(n[0] in (INDEX, SCHEDULE, RESET) for n in notes):   # (a small batch makes its index itself, without queues)
                            check_heads(plan, notes, base)
        # a small batch leaves its schedules out; a forward without the index build makes them up with the options it finds
        for name in ("layer1_order", "large_schedule", "handoff_fences"):
            for other in ("layer1_order", "large_schedule", "handoff_fences"):
                plan.set(other, 0)
            plan.set("phases", 15)
            plan.forward()
            plan.set("phases", 14)
            plan.set(name, 1)
            check_heads(plan, plan.forward())
        plan.close()


def test_queue_heads_do_not_outgrow_the_static_workspace(lib):
    """Just below 32 MiB a plan keeps to the room in the status words; every other one has its heads 256 bytes apart."""
    limit, seen = 32 << 20, set()
    for T in range(30000, 33000):
        plan = Plan(lib, T, 256, 256, 4, 1, act=0, tile_m=256, n_cu=64)   # more than a round
        total = plan.bytes()
        stride = plan.forward()[0][2]
        plan.close()
        assert total % 256 == 0
        if stride == 4:
            assert limit - 4096 < total <= limit
        else:
            assert stride == 256 and not limit < total <= limit + 4096
        seen.add((stride, total <= limit))
    assert seen == {(4, True), (256, True), (256, False)}


@pytest.mark.parametrize("T, H, F, E, k, act, options, rows", [
    (509, 4096, 6400, 16, 2, 1, {}, 256),                       # an expert's only tile
    (509, 4096, 6400, 16, 2, 1, {"tile_m": 64}, 64),            # 64 rows per expert in 64-row tiles: some have two, one after the other
    (1200, 4096, 6400, 16, 2, 1, {"tile_m": 128}, 128),         # two for each
    (1200, 3584, 2560, 64, 8, 1, {"tile_m": 64, "weights_packed": 1}, 64),
    (640, 4096, 1792, 8, 2, 1, {}, 128),                        # 160 rows per expert, 128-row tiles
    (1952, 4096, 6400, 16, 2, 1, {}, 256),                      # 244 rows per expert on average
    (1953, 4096, 6400, 16, 2, 1, {}, 0),
    (448, 4096, 1792, 8, 2, 1, {}, 128),                        # one round of 64-row tiles, two for an expert, run at the same time
    (448, 4096, 1792, 8, 2, 1, {"tile_m": 128}, 128),
    (320, 4096, 2176, 8, 2, 1, {"tile_m": 64}, 64),             # 17 column tiles: no longer one round
    (200, 4096, 1408, 4, 2, 1, {}, 64),                         # 138 MB: the second tile may still find them in the caches
    (200, 4096, 1152, 4, 2, 1, {}, 0),                          # 113 MB
])
def test_weights_are_streamed_for_experts_of_one_tile(lib, T, H, F, E, k, act, options, rows):
    """Whose weights are loaded non-temporally: those nobody fetches again, by the rows of the expert and the height of the tiles."""
    plan = Plan(lib, T, H, F, E, k, act, **options)
    notes = plan.forward()
    assert [n[6] for n in notes if n[0] in (LAYER0, LAYER1)] == [rows, rows]
    plan.close()


@pytest.mark.parametrize("T, H, F, E, k, act, small", [
    (2048, 256, 512, 4, 2, 0, True),       # 4096 pairs, half a MiB per expert: 64 MiB
    (2049, 256, 512, 4, 2, 0, False),
    (512, 1024, 1024, 1, 1, 0, True),      # 4 MiB: 64 MiB at 512 rows
    (513, 1024, 1024, 1, 1, 0, False),
    (1536, 768, 768, 1, 1, 1, False),
    (2048, 512, 256, 5, 2, 1, False),
    (2048, 256, 384, 7, 2, 1, False),
    (2048, 512, 128, 10, 2, 1, True),
    (600, 768, 384, 2, 2, 1, True),
    (64, 1024, 1280, 1, 1, 0, False),      # 5 MiB
    (4097, 256, 256, 1, 1, 0, False),
])
@pytest.mark.parametrize("packed", [0, 1])
def test_small_weights_take_the_small_batch_kernel_while_they_pass_the_cache_often_enough(lib, T, H, F, E, k, act, small, packed):
    plan = Plan(lib, T, H, F, E, k, act, weights_packed=packed)
    kinds = [n[0] for n in plan.forward()]
    assert (DECODE0 in kinds and DECODE1 in kinds) == small
    assert (LAYER0 in kinds and LAYER1 in kinds) == (not small)
    plan.close()


@pytest.mark.parametrize("T, E, k, own", [(384, 24, 1, 1), (385, 25, 1, 0), (192, 4, 2, 1), (193, 4, 2, 0), (96, 64, 4, 1), (97, 64, 4, 0),
                                          (64, 65, 4, 1), (65, 65, 4, 0), (32, 128, 8, 1), (33, 128, 8, 0), (1, 129, 8, 0)])
def test_up_to_how_many_pairs_a_small_batch_makes_its_index_itself(lib, T, E, k, own):
    plan = Plan(lib, T, 256, 256, E, k, act=0, weights_packed=1)
    notes = plan.forward()
    assert [n[5] for n in notes if n[0] in (DECODE0, DECODE1)] == [own, own]
    assert any(n[0] == INDEX for n in notes) == (not own)
    plan.close()
