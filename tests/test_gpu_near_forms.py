"""Near field of one and of several fields: its far, shifted and close forms
against the oracle's direct sum, with every pair in the near field (theta so
small that nothing is accepted), and the work items' edges."""
import numpy as np
import pytest

import meshgen
import oracle

pytestmark = pytest.mark.gpu


def _evaluate(nodes, tets, M, targets, leaf):
    """u [F, n] of M [F, n_nodes, 3]."""
    import torch

    import paper_1606_00247_amd as T

    plan = T.tfmm_plan_create(nodes, tets, targets=targets, p=2, leaf_size=leaf, theta=1e-3)
    assert T.tfmm_plan_stats(plan)["n_m2l"] == 0
    u = T.tfmm_evaluate(plan, torch.from_numpy(np.ascontiguousarray(M)).to("cuda:0")).cpu().numpy()
    T.tfmm_plan_destroy(plan)
    return u


def _close_targets(nodes, tets, eps, rng, n=24):
    """Points eps away from edges, faces and corners (eps 0: on them)."""
    t = tets[rng.integers(0, len(tets), n)]
    lam = rng.uniform(0.1, 0.9, (n, 1))
    x = [nodes[t[:, 0]] * lam + nodes[t[:, 1]] * (1 - lam), nodes[t[:, :3]].mean(axis=1), nodes[t[:, 2]]]
    return np.concatenate([p + eps * rng.uniform(-1, 1, (n, 3)) for p in x])


# The tolerance: the oracle's sum is within 2e-15 of the exact value here and
# the closed form loses about (d / diam)^4 eps, below 1e-12 of the result for
# targets inside the mesh and next to it (d <= 5 diam).
@pytest.mark.parametrize("leaf", [1, 5, 13, 64])
@pytest.mark.parametrize("eps", [0.0, 1e-9, 1e-5, 1e-3, 3e-2, 0.2])
def test_close_targets_vs_oracle(eps, leaf):
    rng = np.random.default_rng(int(1e9 * eps) % 1000 + leaf)
    nodes, tets = meshgen.box_mesh((3, 2, 3), seed=2)
    M = meshgen.random_fields(len(nodes), F=1, seed=9)
    x = _close_targets(nodes, tets, eps, rng)
    u = _evaluate(nodes, tets, M, x, leaf)
    ref = oracle.direct(nodes, tets, M, targets=x)
    assert np.linalg.norm(u - ref) <= 1e-12 * np.linalg.norm(ref)


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 129])
@pytest.mark.parametrize("mesh", ["one", "unjittered"])
def test_work_item_edges_vs_oracle(mesh, n):
    if mesh == "one":
        nodes = np.array([[0.0, 0, 0], [1, 0, 0], [0, 1, 0], [0, 0, 1]])
        tets = np.array([[0, 1, 2, 3]], dtype=np.int32)
    else:  # targets in face planes and on the lines of edges
        nodes, tets = meshgen.box_mesh((2, 2, 1), jitter=0.0)
    M = meshgen.random_fields(len(nodes), F=1, seed=3)
    rng = np.random.default_rng(n)
    x = rng.integers(-2, 5, (n, 3)) / 2.0
    u = _evaluate(nodes, tets, M, x, 64)
    ref = oracle.direct(nodes, tets, M, targets=x)
    assert np.abs(u - ref).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("F", [2, 3, 5, 9, 17, 33])
@pytest.mark.parametrize("eps", [0.0, 1e-9, 1e-3, 0.2])
def test_several_fields_vs_oracle(eps, F):
    """Passes of 2, 4, 8 and 16 fields, full and padded, and a last field alone."""
    rng = np.random.default_rng(F)
    nodes, tets = meshgen.box_mesh((3, 2, 3), seed=2)
    M = meshgen.random_fields(len(nodes), F=F, seed=9)
    x = _close_targets(nodes, tets, eps, rng, n=30)
    u = _evaluate(nodes, tets, M, x, 13)
    ref = oracle.direct(nodes, tets, M, targets=x)
    for f in range(F):
        assert np.linalg.norm(u[f] - ref[f]) <= 1e-12 * np.linalg.norm(ref[f])


@pytest.mark.parametrize("F", [1, 4])
def test_faces_shared_in_odd_ways_vs_oracle(F):
    """Faces of three tets, of two tets on the same side and of a tet listed
    twice: only a face between two tets, one on either side, cancels."""
    nodes = np.array([[0.0, 0, 0], [1, 0, 0], [0, 1, 0], [0, 0, 1], [0.2, 0.2, 0.7], [0.3, 0.3, -0.8], [1.1, 0.9, 0.8]])
    tets = np.array([[0, 1, 2, 3], [0, 1, 2, 4], [0, 2, 1, 5], [1, 2, 3, 6], [1, 2, 3, 6]], dtype=np.int32)
    M = meshgen.random_fields(len(nodes), F=F, seed=5)
    x = np.random.default_rng(1).uniform(-0.5, 1.5, (70, 3))
    u = _evaluate(nodes, tets, M, x, 64).reshape(F, -1)
    ref = oracle.direct(nodes, tets, M, targets=x).reshape(F, -1)
    for f in range(F):
        assert np.linalg.norm(u[f] - ref[f]) <= 1e-12 * np.linalg.norm(ref[f])
