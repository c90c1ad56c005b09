"""Sums over the near-field surrogate's band of pairs on small leaves, where a
target comes up several times among the pairs of one wavefront: against the
oracle's pair integral, pair by pair."""
import numpy as np
import pytest

import meshgen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    return torch, torch.device("cuda:0")


def _mesh(kind):
    return meshgen.box_mesh(3, seed=2) if kind == "box" else meshgen.sphere_mesh(6, seed=3)[:2]


@pytest.fixture(scope="module")
def bands(orc):
    """Per mesh: nodes, tets, M and the exact band potential at the nodes."""
    out = {}
    for kind in ("box", "sphere"):
        nodes, tets = _mesh(kind)
        M = meshgen.random_fields(len(nodes), F=1, seed=5)[0]
        v = nodes[tets]
        size = np.max([np.linalg.norm(v[:, i] - v[:, j], axis=1) for i in range(4) for j in range(i)], axis=0)
        far = np.linalg.norm(nodes[:, None] - v.mean(axis=1)[None], axis=2) / size
        u = np.zeros(len(nodes))
        for i, t in zip(*np.nonzero((far >= 2.0) & (far < 6.0))):
            u[i] += orc.tet_potential(nodes[i], v[t], M[tets[t]])
        out[kind] = nodes, tets, M, u
    return out


# every pair in the near field (nothing is accepted at this theta)
@pytest.mark.parametrize("leaf", [1, 2, 8, 16, 64])
@pytest.mark.parametrize("kind", ["box", "sphere"])
def test_band_potential(torch_dev, bands, kind, leaf):
    import paper_1606_00247_amd as T

    torch, dev = torch_dev
    nodes, tets, M, ref = bands[kind]
    plan = T.tfmm_plan_create(nodes, tets, p=2, leaf_size=leaf, theta=1e-3)
    print("band", kind, leaf, flush=True)
    u = T.tfmm_band_potential(plan, torch.from_numpy(M).to(dev), False).cpu().numpy()
    # the closed form loses up to 6^4 eps a pair, here of pairs of one size
    assert np.abs(u - ref).max() <= 1e-11 * np.abs(ref).max()


@pytest.mark.parametrize("F", [1, 3])
@pytest.mark.parametrize("leaf", [1, 8, 16])
def test_gauss_rule_in_the_band(torch_dev, bands, leaf, F):
    """Evaluation with the 27-point rule (degree 5) for the band's pairs: its error
    falls as (distance / diameter)^-6, up to 3e-4 of a pair 2 diameters apart; some
    fifty of these, of random sign and each below 1% of the largest potential."""
    import paper_1606_00247_amd as T

    torch, dev = torch_dev
    nodes, tets, _, _ = bands["sphere"]
    M = torch.from_numpy(meshgen.random_fields(len(nodes), F=F, seed=6)).to(dev)
    plan = T.tfmm_plan_create(nodes, tets, p=2, leaf_size=leaf, theta=1e-3)
    exact = T.tfmm_evaluate(plan, M)
    T.tfmm_plan_set_surrogate(plan, T.SUR_GAUSS)
    print("gauss band", leaf, F, flush=True)
    u = T.tfmm_evaluate(plan, M)
    assert float((u - exact).abs().max()) <= 5e-5 * float(exact.abs().max())
