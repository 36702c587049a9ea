"""Plan statistics against what the launches do."""
import pytest

pytestmark = pytest.mark.gpu


def test_top_pairs_are_those_of_the_fp32_form():
    """Only the FP32 form has levels of its own in FP64; the FP64 form runs every pair in the
    main M2L launch, whose rate is priced by the pairs that are not top pairs."""
    from paper_1908_10863_amd import fmmlm as F, workloads as W
    w = W.config(0, n=4000)
    top = {}
    for precision in (F.FMMLM_FP64, F.FMMLM_FP32_COMPENSATED):
        plan = F.Plan(w["d"], w["eps"], w["x"], w["y"], w["z"], w["layer"], p=4, leaf_cap=10, precision=precision)
        st = plan.stats()
        plan.close()
        top[precision] = st["m2l_top_pairs"]
        pairs = st["m2l_free_pairs"] + st["m2l_reaction_pairs"]
    assert top[F.FMMLM_FP64] == 0
    assert 0 < top[F.FMMLM_FP32_COMPENSATED] < pairs
