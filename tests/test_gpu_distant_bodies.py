"""Near field of bodies that lie far apart in one leaf: a body's potential keeps
its digits, whatever else the leaf holds."""
import numpy as np
import pytest

import meshgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F", [1, 2, 5, 17])
@pytest.mark.parametrize("gap", [300.0, 30000.0])
def test_two_bodies_in_one_leaf(F, gap):
    """Each body's own potential beside a body without magnetisation and alone."""
    import torch
    assert torch.cuda.is_available()

    import paper_1606_00247_amd as T

    a, ta = meshgen.box_mesh(1, seed=1)  # twelve tets of sixteen nodes in all
    b, tb = meshgen.box_mesh(1, seed=2)
    b = np.round(b * 2.0 ** 30) / 2.0 ** 30 + gap * np.array([1.0, 0.5, 0.25])  # exact
    na, n = len(a), len(a) + len(b)
    M = meshgen.random_fields(n, F=F, seed=3)

    def run(nodes, tets, M):
        plan = T.tfmm_plan_create(nodes, tets, p=2, leaf_size=300, theta=1e-3)
        u = T.tfmm_evaluate(plan, torch.from_numpy(np.ascontiguousarray(M)).cuda()).cpu().numpy().reshape(F, -1)
        T.tfmm_plan_destroy(plan)
        return u

    both = np.concatenate([a, b]), np.concatenate([ta, tb + na]).astype(np.int32)
    for name, own, nodes, tets in (("first", slice(0, na), a, ta), ("second", slice(na, n), b, tb)):
        print("distant bodies", F, gap, name, flush=True)
        m = np.zeros_like(M)
        m[:, own] = M[:, own]
        u, alone = run(*both, m)[:, own], run(nodes, tets, M[:, own])
        # a few dozen roundings of the potential, of the distances and of positions within
        # a chunk (up to some thirty sizes of a tet)
        assert np.abs(u - alone).max() <= 1e-13 * np.abs(alone).max(), (name, np.abs(u - alone).max())
