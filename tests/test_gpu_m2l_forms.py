"""M2L in FP32 and split BF16 against the packed FP64 form: field counts at the
edges of the groups of 16 and of pairs of groups, orders on both sides of the
register limits, trees with and without translations between levels."""
import numpy as np
import pytest

import meshgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,leaf,F", [(1, 4, 2), (2, 9, 17), (3, 4, 1), (4, 16, 5), (6, 9, 33), (8, 8, 3), (8, 30, 16), (8, 9, 48),
                                      (9, 9, 32), (10, 20, 7), (10, 9, 49)])
def test_reduced_precisions_vs_fp64(p, leaf, F):
    import torch

    import paper_1606_00247_amd as T

    nodes, tets = meshgen.box_mesh((6, 5, 4), seed=p + leaf)
    tets = tets[np.abs(nodes[tets].mean(1) - nodes.mean(0)).sum(1) > 0.9]  # uneven: translations between levels
    M = torch.from_numpy(meshgen.random_fields(len(nodes), F=F, seed=F)).to("cuda:0")
    plan = T.tfmm_plan_create(nodes, tets, p=p, leaf_size=leaf, theta=0.6)
    one = [T.tfmm_evaluate(plan, M[f].contiguous()).cpu().numpy().ravel() for f in range(F)]
    # FP64 to rounding; the others as the accuracy of their operands allows (2^-24 and 2^-16 a
    # term, sums in FP32)
    for prec, tol in ((T.M2L_FP64, 1e-12), (T.M2L_FP32, 2e-6), (T.M2L_BF16X3, 1e-5), (T.M2L_BF16X6, 2e-6)):
        T.tfmm_plan_set_m2l_precision(plan, prec)
        u = T.tfmm_evaluate(plan, M).cpu().numpy().reshape(F, -1)
        for f in range(F):
            assert np.linalg.norm(u[f] - one[f]) <= tol * np.linalg.norm(one[f]), (prec, f)
    T.tfmm_plan_destroy(plan)
