"""The gate against the oracle: every way experts fall into a wavefront's lanes, ties (among them 0 and -0), masked experts (minus
infinity, the type's lowest value), infinities; rows with a NaN do not disturb the others."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,k", [(1, 1), (2, 2), (8, 2), (63, 8), (64, 8), (64, 64), (65, 17), (128, 1), (200, 16), (256, 64)])
def test_gate(E, k):
    import paper_2502_19811_amd as moe
    rng = np.random.default_rng(E * 100 + k)
    T = 203
    x = rng.standard_normal((T, E)).astype(np.float32)
    x[1::5] = np.round(x[1::5])                                    # ties, and both zeros
    x[2::5] *= np.where(rng.random((T, E)) < 0.5, 0.0, -0.0)[2::5].astype(np.float32)
    lowest = np.float32(np.finfo(np.float32).min)
    mask = rng.random((T, E)) < 0.6
    mask[np.arange(T), rng.integers(0, E, T)] = False              # something is left
    x[3::5] = np.where(mask, lowest, x)[3::5]
    x[4::5] = np.where(mask, -np.inf, x)[4::5]
    x[0, rng.integers(0, E)] = lowest
    ids_ref, w_ref = orc.route_topk(x, k)
    clean = torch.from_numpy(x).cuda()
    ids = torch.full((T, k), -7, dtype=torch.int32, device="cuda")
    w = torch.full((T, k), -7.0, device="cuda")
    print(f"gate E {E} k {k}", flush=True)
    moe.moe_route_topk(clean, k, ids, w)
    np.testing.assert_array_equal(ids.cpu().numpy(), ids_ref)
    # fp32 exp, sum and quotient: a few units in the last place of numbers up to 1
    np.testing.assert_allclose(w.cpu().numpy(), w_ref, rtol=1e-5, atol=1e-6)

    broken = clean.clone()
    broken[7::11, E // 2] = float("nan")
    ids2, w2 = torch.full_like(ids, -7), torch.full_like(w, -7.0)
    moe.moe_route_topk(broken, k, ids2, w2)
    rest = torch.ones(T, dtype=torch.bool)
    rest[7::11] = False
    assert torch.equal(ids2.cpu()[rest], ids.cpu()[rest]) and torch.equal(w2.cpu()[rest], w.cpu()[rest])
    # plus infinity beats everything: one is taken first, its weight is not defined (inf - inf)
    top = clean.clone()
    at = torch.from_numpy(rng.integers(0, E, T)).cuda()
    top[torch.arange(T, device="cuda"), at] = float("inf")
    moe.moe_route_topk(top, k, ids2, w2)
    assert torch.equal(ids2[:, 0].long(), at)
