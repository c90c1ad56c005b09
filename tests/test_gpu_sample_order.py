"""Training samples of the near-field surrogate with a seed: the pairs drawn are
pinned (the first four of their inputs), so that a network
trained with a seed stays the network of that seed."""
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

PINNED = {
    (6, 16, 11): [[-0.432693, -0.895712, -0.102351, -0.120983], [0.190224, -0.907938, 0.373449, -0.052218],
                  [0.669106, -0.203219, 0.714842, -0.338921], [0.070419, -0.070205, 0.995044, -0.441443],
                  [-0.760181, 0.641805, -0.10105, -0.30778], [0.057342, -0.114699, -0.991744, -0.425605]],
    (5, 8, 7): [[-0.818978, -0.419362, -0.391676, -0.421229], [-0.817243, -0.441306, -0.370626, -0.162199],
                [-0.652846, 0.469418, 0.594507, -0.322305], [-0.453048, 0.885885, -0.099773, -0.433785],
                [-0.072444, 0.975295, -0.208692, -0.120542], [-0.146574, 0.722725, 0.675414, -0.520883]],
}


@pytest.mark.parametrize("n,leaf,seed", sorted(PINNED))
def test_seeded_samples(torch_dev, n, leaf, seed):
    import paper_1606_00247_amd as T

    nodes, tets = meshgen.box_mesh(n, seed=2)
    plan = T.tfmm_plan_create(nodes, tets, p=4, leaf_size=leaf, theta=0.5)
    print("samples", n, leaf, seed, flush=True)
    X, _ = T.tfmm_surrogate_samples(plan, 6, seed=seed)
    assert np.abs(X[:, :4] - np.array(PINNED[n, leaf, seed])).max() <= 2e-6  # six digits of FP32 numbers
