"""Every launch variant of the FP32 M2L gives the same bits, at each order that has
variants, on units below the FP64 top levels (stats: m2l_chunks > 0) and in the batched
form.  The variants differ in how many k-steps of an operator go through LDS at once, in
reserved LDS and in the order of the boxes, never in the order of the sums."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [8, 9, 10])
@pytest.mark.parametrize("g", [1, 17])
def test_variants_are_bit_equal(p, g):
    import torch
    from paper_1908_10863_amd import fmmlm as F, workloads as W
    w = W.make_layered((0.0, -1.0), (1.0, 5.0, 2.0), W.split_even(4001, 3), 6, nrhs=g)
    q = torch.tensor(w["q"], device="cuda")
    plan = F.Plan(w["d"], w["eps"], w["x"], w["y"], w["z"], w["layer"], p=p, leaf_cap=12, mac_d2=4,
                  precision=F.FMMLM_FP32_COMPENSATED, max_rhs=g)
    assert plan.stats()["m2l_chunks"] > 0
    if g > 1:
        plan.set_variants(batch_min=2)
    ref = plan.eval(q)
    for v in range(6 if g == 1 else 10):
        plan.set_variants(**{"m2l" if g == 1 else "batch": v})
        assert torch.equal(plan.eval(q), ref), v
    plan.close()
