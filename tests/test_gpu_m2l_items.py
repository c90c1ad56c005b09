"""Work items of the packed M2L: cut for the evaluation that runs, whatever ran
on the plan before."""
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


def _plan(n=9, p=4, leaf=8, **k):
    import paper_1606_00247_amd as T

    nodes, tets = meshgen.box_mesh(n, seed=1)
    return T, nodes, T.tfmm_plan_create(nodes, tets, p=p, leaf_size=leaf, theta=0.5, **k)


def _evaluate(torch_dev, T, plan, nodes, F):
    torch, dev = torch_dev
    M = meshgen.random_fields(len(nodes), F=F, seed=3)
    return T.tfmm_evaluate(plan, torch.from_numpy(M).to(dev)).cpu().numpy()


def test_field_counts_in_turn(torch_dev):
    """A plan that saw F = 13 before F = 1 holds the same lists as one that saw them the other way round."""
    held, u = [], []
    for order in ((13, 1), (1, 13), (1, 13, 1, 13)):
        T, nodes, plan = _plan()
        assert T.tfmm_plan_stats(plan)["n_m2l"] * 13 // 16 > 2 * 48 * 512  # enough groups for longer items
        for F in order:
            print("field counts", order, F, flush=True)
            v = _evaluate(torch_dev, T, plan, nodes, F)
            if F == 13:
                u.append(v)
        held.append(T.tfmm_plan_stats(plan)["device_bytes"])
        T.tfmm_plan_destroy(plan)
    assert held[0] == held[1] == held[2]
    for v in u[1:]:
        assert np.abs(v - u[0]).max() <= 1e-13 * np.abs(u[0]).max()
