"""Limits of a plan's operator tables."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_many_operators_at_the_largest_order(oracle_mod):
    """Seven interfaces give 196 reaction components and more than 29,000 M2L operators at
    p = 16, which share about 8,000 frame operators: their tables (380 KB each in FP64) are
    far below the 32 GiB a plan may take for them, and the plan is made.  Against the direct
    sum, within the FP32 form's 1e-5."""
    import torch
    from paper_1908_10863_amd import fmmlm as F, workloads as W
    d = [-1.0 * i for i in range(7)]
    eps = list(np.random.default_rng(7).uniform(1.0, 12.0, 8))
    n = 8 * 260
    w = W.make_layered(d, eps, W.split_even(n, 8), 33)
    plan = F.Plan(w["d"], w["eps"], w["x"], w["y"], w["z"], w["layer"], p=16, leaf_cap=20,
                  precision=F.FMMLM_FP32_COMPENSATED, mac_d2=6)
    st = plan.stats()
    print(f"{st['n_sommerfeld_tasks']} tasks, {st['n_trees']} trees, {st['device_bytes'] / 2 ** 30:.1f} GiB", flush=True)
    assert st["n_reaction_ops"] > 29000 and st["n_sommerfeld_tasks"] < 10000
    phi = plan.eval(torch.tensor(w["q"][0], device="cuda")).cpu().numpy()
    plan.close()
    t = np.arange(0, n, 52)
    ref = oracle_mod.potential(d, eps, w["x"], w["y"], w["z"], w["layer"], w["q"][0], targets=t, method="quad")
    assert np.linalg.norm(phi[t] - ref) <= 1e-5 * np.linalg.norm(ref)
