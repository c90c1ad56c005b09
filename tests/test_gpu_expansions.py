"""Multipole and local expansions of every cell against the oracle, at every
order and at the edges of the kernels' tiles: leaves of fewer and of more tets
than a matrix-core step or a stage takes, field chunks full and cut short."""
import numpy as np
import pytest

import meshgen
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,leaf,F", [(1, 3, 1), (2, 1, 3), (3, 17, 4), (4, 16, 2), (5, 64, 5), (6, 5, 1), (7, 33, 1),
                                      (8, 12, 6), (8, 70, 1), (9, 20, 3), (10, 9, 1), (10, 65, 7)])
def test_expansions_vs_oracle(p, leaf, F):
    import torch

    import paper_1606_00247_amd as T

    nodes, tets = meshgen.box_mesh((5, 4, 5), seed=p)
    M = meshgen.random_fields(len(nodes), F=F, seed=p + 1)
    plan = T.tfmm_plan_create(nodes, tets, p=p, leaf_size=leaf, theta=0.6)
    u = T.tfmm_evaluate(plan, torch.from_numpy(M).to("cuda:0")).cpu().numpy()
    ref = oracle.FMM(nodes, tets, p, leaf, 0.6)
    v = ref.evaluate(M)
    for f in range(F):
        assert np.linalg.norm(u[f] - v[f]) <= 1e-12 * np.linalg.norm(v[f])
    ref.evaluate(M[-1])  # the expansions kept are the last field's
    cells, _ = T.tfmm_plan_cells(plan)
    other, _ = ref.cells()
    at = {tuple(c[:4]): i for i, c in enumerate(other)}
    order = np.array([at[tuple(c[:4])] for c in cells])
    for which, count in (("Q", 4), ("L", 5)):
        g, o = T.tfmm_plan_expansions(plan, which), ref.expansions(which)[order]
        used = cells[:, count] > 0
        scale = np.abs(o).max(axis=1)
        if which == "L":
            # a cell's local is a sum over hundreds of source cells and may cancel: one
            # rounding of the field moves a cell of the first case, 4000 times smaller
            # than its neighbours, by 2.3e-12 of itself in the oracle.  Roundings are
            # relative to the terms, which have the size of the level's locals.
            for lv in np.unique(cells[used, 0]):
                at_level = used & (cells[:, 0] == lv)
                scale[at_level] = scale[at_level].max()
        assert (np.abs(g - o).max(axis=1)[used] <= 1e-12 * scale[used]).all(), which
    T.tfmm_plan_destroy(plan)
