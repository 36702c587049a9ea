"""The FP64 free-space near field in both of its unit sizes: 64 targets where the launch
would end on its longest unit of 128 (more than 1.3 times a CU's share of the pairs) or no
leaf holds more than 64 charges, 128 elsewhere.  Against the direct sum at sampled targets,
by the bound that p = 12 at the default acceptance has elsewhere (1e-7: truncation)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _side(plan):
    """(64 or 128, largest leaf) by the rule, from the plan's own lists."""
    boxes, pf = plan.lists(0).astype(np.int64), plan.lists(2).astype(np.int64)
    start, count = boxes[:, 0], boxes[:, 1]
    leaf, s0, sn = pf[:, 0], pf[:, 1], pf[:, 2]
    later = np.bincount(leaf, weights=np.where(s0 >= start[leaf], sn, 0), minlength=len(boxes))
    used = np.unique(leaf)
    work, longest = (count * later)[used].sum(), (np.minimum(count, 128) * later)[used].max()
    largest = count[used].max()
    return (64 if largest <= 64 or 256 * longest > 1.3 * work else 128), largest


@pytest.mark.parametrize("n,cap,units", [(2400, 220, 64), (12000, 192, 64), (20000, 64, 64), (85000, 192, 128)])
def test_fp64_near_field_by_unit_size(n, cap, units, oracle_mod):
    import torch
    from paper_1908_10863_amd import fmmlm as F, workloads as W
    w = W.make_layered((0.0,), (1.0, 5.0), W.split_even(n, 2), 8)
    plan = F.Plan(w["d"], w["eps"], w["x"], w["y"], w["z"], w["layer"], p=12, leaf_cap=cap, mac_d2=6)
    assert _side(plan)[0] == units and (_side(plan)[1] > 64) == (cap > 64)
    q = torch.tensor(w["q"][0], device="cuda")
    phi = plan.eval(q).cpu().numpy()
    assert np.array_equal(plan.eval(q).cpu().numpy(), phi)
    plan.close()
    t = np.sort(np.random.default_rng(2).choice(n, 64, replace=False))
    ref = oracle_mod.potential(w["d"], w["eps"], w["x"], w["y"], w["z"], w["layer"], w["q"][0], targets=t)
    assert np.linalg.norm(phi[t] - ref) <= 1e-7 * np.linalg.norm(ref)
