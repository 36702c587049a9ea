"""The FP64 form's M2L matrix-core kernel over every wave grid it has (one per number of
16-row blocks of (p+1)^2) and over ragged chunks: few targets, many charges per leaf and
an odd number of them.  Against the direct sum, by the truncation bound of the order and
acceptance: the far field decays like (0.87 / 2)^p at acceptance 6 (boxes of radius 0.87 at
distance sqrt 6 and more), times 10 for the sum over terms and boxes, plus 1e-12 of rounding.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [2, 4, 5, 6, 8, 9, 10, 11, 12, 13, 14, 15, 16])
@pytest.mark.parametrize("n,cap", [(3001, 5), (777, 2)])
def test_fp64_chunks_against_the_direct_sum(p, n, cap, oracle_mod):
    import torch
    from paper_1908_10863_amd import fmmlm as F, workloads as W
    w = W.config(0, n=n)
    q = torch.tensor(w["q"][0], device="cuda:0")
    t = np.arange(0, n, n // 50)
    ref = oracle_mod.potential(w["d"], w["eps"], w["x"], w["y"], w["z"], w["layer"], w["q"][0], targets=t)
    plan = F.Plan(w["d"], w["eps"], w["x"], w["y"], w["z"], w["layer"], p=p, leaf_cap=cap)
    assert plan.stats()["m2l_chunks"] > 0
    phi = plan.eval(q).cpu().numpy()[t]
    plan.close()
    err = np.linalg.norm(phi - ref) / np.linalg.norm(ref)
    assert err <= 10 * 0.435 ** p + 1e-12, (p, err)


@pytest.mark.parametrize("p", [1, 2, 3, 4, 5, 7, 8, 10, 11, 12, 13, 14, 15, 16])
@pytest.mark.parametrize("g", [2, 17, 33])
def test_batched_fp32_against_fp64_per_vector(p, g):
    """The batched FP32 form's M2L (one block per target box) over every number of row
    blocks, from one batch of k-steps an entry on, with a partly filled group of 16
    vectors.  Against the FP64 form vector by vector: the same truncation, so the
    difference is FP32 rounding of sums of at most 153 terms of size 1 (2^-24 each,
    adding up like their square root, 7.4e-7) times 3."""
    import torch
    from paper_1908_10863_amd import fmmlm as F, workloads as W
    n = 4001
    w = W.make_layered((0.0, -0.6, -1.4), (1.0, 3.9, 11.7, 2.5), W.split_even(n, 4), 3, nrhs=g)
    q = torch.tensor(w["q"], device="cuda:0")
    kw = dict(p=p, leaf_cap=12, mac_d2=4, max_rhs=g)
    out = []
    for precision, width in ((0, g + 1), (1, 2)):
        plan = F.Plan(w["d"], w["eps"], w["x"], w["y"], w["z"], w["layer"], precision=precision, **kw)
        plan.set_variants(batch_min=min(width, 64))
        out.append(plan.eval(q))
        plan.close()
    err = ((out[1] - out[0]).norm() / out[0].norm()).item()
    assert err <= 3 * 7.4e-7, (p, g, err)
