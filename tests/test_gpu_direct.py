"""Direct sum against the oracle's at the edges of its kernel: blocks of tets
full and cut short, one target and counts around a workgroup's 256, field
chunks full, padded and repeated, targets in every distance class."""
import numpy as np
import pytest

import meshgen
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("box,n,F", [((1, 1, 1), 1, 1), ((1, 1, 1), 255, 2), ((2, 2, 1), 256, 3), ((3, 2, 1), 257, 5),
                                     ((3, 3, 2), 700, 9), ((2, 3, 3), 64, 17), ((4, 4, 4), 1100, 1)])
def test_direct_vs_oracle(box, n, F):
    import torch

    import paper_1606_00247_amd as T

    nodes, tets = meshgen.box_mesh(box, seed=n)
    M = meshgen.random_fields(len(nodes), F=F, seed=F)
    rng = np.random.default_rng(n + F)
    x = nodes[rng.integers(0, len(nodes), n)]
    # a third at nodes, the others up to 50 extents away
    x = x + rng.standard_normal((n, 3)) * np.ptp(nodes) * rng.choice([0.0, 0.3, 1, 3, 8, 50], (n, 1))
    plan = T.tfmm_plan_create(nodes, tets, targets=x, p=2, leaf_size=8, theta=0.5)
    u = T.tfmm_direct(plan, torch.from_numpy(M).to("cuda:0")).cpu().numpy()
    v = np.stack([oracle.direct(nodes, tets, M[f], targets=x) for f in range(F)])
    # of the value of each field over all targets: closed forms within 3 longest edges lose
    # up to 3^4 roundings of a tet's largest term, the far rules 3e-14 of theirs
    for f in range(F):
        assert np.abs(u[f] - v[f]).max() <= 1e-12 * np.abs(v[f]).max()
    T.tfmm_plan_destroy(plan)
