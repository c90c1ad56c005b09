"""Near field of targets next to a tet and of targets far from it that share a
wavefront: the far ones keep the far form's digits.  Uniform fields against
surface charges in extended precision."""
import numpy as np
import pytest

from tests.test_gpu_flat_tets import EPS, _uniform

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F", [1, 2, 5, 16])
@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 0.3, 0.3), (1, 1, 0.2)])
def test_far_beside_close(F, shape):
    import torch
    assert torch.cuda.is_available()

    import paper_1606_00247_amd as T

    rng = np.random.default_rng(4)
    v = np.cumsum(np.concatenate([np.zeros((1, 3)), np.diag(shape)]), axis=0) + rng.uniform(-0.03, 0.03, (4, 3)) * min(shape)
    lam = rng.dirichlet(np.ones(3), 40)
    way = rng.standard_normal((200, 3))
    far = v.mean(axis=0) + way / np.linalg.norm(way, axis=1)[:, None] * rng.uniform(30.0, 100.0, (200, 1))
    # next to its faces and edges; the targets' order in the plan mixes them with the others
    x = np.concatenate([far, lam @ v[:3] + 1e-3, lam @ v[1:] - 1e-3, v[0] + (v[3] - v[0]) * lam[:, :1] + 1e-4])
    m = rng.standard_normal((F, 3))
    M = np.repeat(m[:, None], 4, axis=1)
    plan = T.tfmm_plan_create(v, np.array([[0, 1, 2, 3]], np.int32), targets=x, theta=1e-3, leaf_size=64, p=2)
    assert T.tfmm_plan_stats(plan)["n_m2l"] == 0
    print("mixed targets", shape, F, flush=True)
    u = T.tfmm_evaluate(plan, torch.from_numpy(M if F > 1 else M[0]).cuda()).cpu().numpy().reshape(F, -1)
    T.tfmm_plan_destroy(plan)
    for f in range(F):
        ref, size = _uniform(v, np.array([[0, 1, 2, 3]]), m[f], far)
        # the sum of the faces' terms, of about twenty roundings each (64 allowed)
        worst = float((np.abs(u[f, :200] - ref) / size).max())
        assert worst <= 64 * EPS, (f, worst / EPS)
