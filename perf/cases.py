"""The work this library is used for, as cases that can be timed and compared: gate and layer forward through the
public entry points (moe_route_topk, then moe_layer_forward or moe_layer_forward_static), from a single decoded token
to the largest batch of the workloads, with packed and plain weights, SwiGLU and GELU, resident input and ready flags.

A case is a dict of plain values:
  T, H, F, E, k   tokens, embedding size, expert hidden size, experts, experts per token
  S               source segments of the receive buffer
  act             "swiglu" or "gelu"
  packed          the weights were re-laid out once with moe_pack_weights
  flags           the forward is given ready flags (every segment has arrived)
  zipf            > 0: expert popularity (e + 1)^-zipf is added to the gate logits, and the segments are unequal
  static          moe_layer_forward_static (the library's own workspace) instead of a caller's workspace
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2502_19811_amd as moe

# Expert shapes of workloads.py: (H, F, E, k, largest T of the workload)
_SHAPES = {
    "tiny": (256, 512, 4, 2, 4096),
    "mixtral": (4096, 14336, 8, 2, 32768),
    "mixtral_tp2": (4096, 7168, 8, 2, 16384),
    "mixtral_tp4": (4096, 3584, 8, 2, 16384),
    "mixtral_tp8": (4096, 1792, 8, 2, 16384),
    "qwen2": (3584, 2560, 64, 8, 8192),
    "qwen2_table2": (2048, 1408, 64, 4, 16384),
    "phi35": (4096, 6400, 16, 2, 16384),
}


def _case(shape, T, name=None, S=8, act="swiglu", packed=True, flags=False, zipf=0.0, static=False):
    H, F, E, k, _ = _SHAPES[shape]
    c = dict(T=T, H=H, F=F, E=E, k=k, S=S, act=act, packed=packed, flags=flags, zipf=zipf, static=static)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest layer, on the library's own workspace: launches and latency are everything
        _case("tiny", 128, "tiny_gelu_static", act="gelu", packed=False, static=True),
        # one sequence decoding: one row for each of two experts, the weights are read once for it
        _case("mixtral", 1, "decode_1_mixtral", S=1),
        # a small decode batch: every expert is needed for a few rows
        _case("mixtral", 16, "decode_16_mixtral"),
        # decode batch over many small experts (about 6 rows each)
        _case("qwen2", 48, "decode_48_qwen2"),
        # decode batch on a tensor-parallel slice whose weights were never re-laid out
        _case("mixtral_tp8", 33, "decode_33_tp8_plain", packed=False),
        # a short prompt or a prefill chunk, of an odd length: tens of rows for each expert
        _case("phi35", 509, "chunk_509_phi35"),
        # a prefill chunk on a tensor-parallel slice, plain weights, waiting on ready flags
        _case("mixtral_tp4", 2047, "chunk_2047_tp4_plain_flags", packed=False, flags=True),
        # prefill over many small experts: two M-tiles for each
        _case("qwen2_table2", 8192, "prefill_8192_qwen2_table2"),
        _case("qwen2", 4096, "prefill_4096_qwen2"),
        # prefill with a receive buffer filled by peers: the forward is given ready flags
        _case("phi35", 16384, "prefill_16384_phi35_flags", flags=True),
        # the benchmark's layer
        _case("mixtral", 8192, "prefill_8192_mixtral"),
        # the largest batch, experts and segments unequal
        _case("mixtral", 32768, "prefill_32768_skewed", zipf=1.2),
    ]


def draw(rng):
    """One more case: a shape, any number of tokens up to the shape's largest (even over the logarithm), and the
    options, the usual ones more often than the others."""
    shape = rng.choice(sorted(_SHAPES))
    T = int(round(math.exp(rng.uniform(0.0, math.log(_SHAPES[shape][4])))))
    act = "gelu" if shape == "tiny" or (_SHAPES[shape][1] % 256 == 0 and rng.random() < 0.15) else "swiglu"
    return _case(shape, T, S=rng.choice((1, 2, 5, 8, 8, 8)), act=act, packed=rng.random() < 0.7,
                 flags=rng.random() < 0.25, zipf=1.2 if rng.random() < 0.25 else 0.0, static=shape == "tiny")


def _segments(case, seed):
    T, S = case["T"], case["S"]
    if case["zipf"] > 0:
        p = np.random.default_rng(seed).dirichlet(np.ones(S))
        cuts = np.round(np.cumsum(p)[:-1] * T).astype(int)
    else:
        cuts = [T * s // S for s in range(1, S)]
    return [0, *[int(c) for c in cuts], T]


class _Layer:
    """What a program keeps for one layer: plan, weights, workspace, and the buffers of one batch."""

    def __init__(self, case, seed):
        T, H, F, E, k = (case[n] for n in ("T", "H", "F", "E", "k"))
        self.k, self.flags, self.static = k, case["flags"], case["static"]
        self.act = moe.MOE_ACT_SWIGLU if case["act"] == "swiglu" else moe.MOE_ACT_GELU
        F1 = 2 * F if case["act"] == "swiglu" else F
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)

        def normal(shape, std, dtype):
            return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=g)

        self.x = normal((T, H), 1.0, torch.bfloat16)
        self.W1 = normal((E, H, F1), H ** -0.5, torch.bfloat16)
        self.W2 = normal((E, F, H), F ** -0.5, torch.bfloat16)
        self.logits = normal((T, E), 1.0, torch.float32)
        if case["zipf"] > 0:
            pop = torch.arange(1, E + 1, dtype=torch.float32, device="cuda") ** -case["zipf"]
            self.logits += torch.log(pop / pop.sum())
        self.plan = moe.moe_plan_create(T, H, F, E, k, case["S"], self.act, _segments(case, seed))
        if case["packed"]:
            W1, W2 = torch.empty_like(self.W1), torch.empty_like(self.W2)
            moe.moe_pack_weights(self.plan, self.W1, self.W2, W1, W2)
            self.W1, self.W2 = W1, W2
            moe.moe_plan_set_option(self.plan, "weights_packed", 1)
        self.seg_ready = torch.ones(case["S"], dtype=torch.int32, device="cuda") if self.flags else None
        self.ids = torch.zeros((T, k), dtype=torch.int32, device="cuda")
        self.w = torch.zeros((T, k), dtype=torch.float32, device="cuda")
        self.out = torch.zeros((T, H), dtype=torch.bfloat16, device="cuda")
        self.workspace = None
        if not self.static:
            self.workspace = torch.zeros(moe.moe_plan_workspace_bytes(self.plan), dtype=torch.uint8, device="cuda")

    def __del__(self):
        if getattr(self, "plan", None) is not None:
            moe.moe_plan_destroy(self.plan)


def prepare(case, seed):
    return _Layer(case, seed)


def run(s):
    """Gate, then the layer, on the current stream."""
    moe.moe_route_topk(s.logits, s.k, s.ids, s.w)
    if s.static:
        moe.moe_layer_forward_static(s.plan, s.x, s.ids, s.w, s.W1, s.W2, s.act, s.out, s.seg_ready, 1)
    else:
        moe.moe_layer_forward(s.plan, s.x, s.ids, s.w, s.W1, s.W2, s.act, s.out, s.workspace, s.seg_ready, 1)
    return {"ids": s.ids, "weights": s.w, "out": s.out}


def work(case):
    """Logits, rows, the weights of the experts that some token picks (as many as even routing picks), and the
    outputs; the products of both layers."""
    T, H, F, E, k = (case[n] for n in ("T", "H", "F", "E", "k"))
    F1 = 2 * F if case["act"] == "swiglu" else F
    experts = E * (1.0 - (1.0 - k / E) ** T)
    weights = experts * (H * F1 + F * H) * 2
    rows = 2 * T * H * 2
    gate = T * E * 4 + T * k * 8
    return {"bytes": int(weights + rows + gate), "flops": 2.0 * T * k * (H * F1 + F * H)}


def tolerance(case):
    """The inputs, h, Y and out are bf16, sums fp32.  Against the layer in 64 bits the output is off by 2.35e-3 in the
    2-norm (the same at every size) and by up to 1.45e-2 in one element; four times that is allowed."""
    return {"rel": 9.4e-3, "max": 5.8e-2}
