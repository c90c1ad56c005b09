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


def test_level_lists_cut_by_their_own_translations(torch_dev):
    """With orders per level every level's list is cut by the translations of
    that level: where none has enough for more than 48 groups an item, the
    largest cap and a cap of 48 give the same items."""
    T, nodes, plan = _plan(10)
    pairs = T.tfmm_plan_lists(plan, "m2l")[:, 0]
    level, total = np.bincount(pairs).max(), len(pairs)
    F = [f for f in range(1, 16, 2) if level * f // 16 // 512 <= 48 and total * f // 16 // 512 >= 50]
    assert F, (level, total)
    T.tfmm_plan_set_level_orders(plan, [4] * T.tfmm_plan_stats(plan)["depth"] + [3])
    held = []
    for cap in (4096, 48):
        T.tfmm_plan_set_schedule(plan, 256, 0, 1, cap)
        print("level lists", cap, F[0], flush=True)
        _evaluate(torch_dev, T, plan, nodes, F[0])
        held.append(T.tfmm_plan_stats(plan)["device_bytes"])
    assert held[0] == held[1]


def test_autotune_leaves_equal_schedules_alone(torch_dev):
    """On a small mesh every cap gives the same items: tuning times them once
    and keeps the plan's cap."""
    for _ in range(6):
        T, nodes, plan = _plan(5, 3, 16)
        cap = T.tfmm_plan_stats(plan)["m2l_groups_per_item"]
        T.tfmm_plan_autotune(plan)
        assert T.tfmm_plan_stats(plan)["m2l_groups_per_item"] == cap
        T.tfmm_plan_destroy(plan)
