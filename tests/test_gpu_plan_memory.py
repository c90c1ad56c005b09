"""Device memory of a plan: the records that only evaluations of several fields
read are allocated by the first of these."""
import pytest

import meshgen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    return torch, torch.device("cuda:0")


def _fields(torch_dev, n, F):
    torch, dev = torch_dev
    return torch.from_numpy(meshgen.random_fields(n, F=F, seed=3)).to(dev), \
        torch.empty((F, n), dtype=torch.float64, device=dev)


def _held(T, plan):
    return T.tfmm_plan_stats(plan)["device_bytes"]


def test_records_of_several_fields_on_demand(torch_dev):
    """Plans that evaluate one field, or apply a stored near field, do not hold
    the tets' records for several fields (over 500 bytes a tet)."""
    import paper_1606_00247_amd as T

    nodes, tets = meshgen.box_mesh(12, seed=1)
    plan = T.tfmm_plan_create(nodes, tets, p=2, leaf_size=64, theta=0.5)
    M1, u1 = _fields(torch_dev, len(nodes), 1)
    M2, u2 = _fields(torch_dev, len(nodes), 2)
    T.tfmm_evaluate(plan, M1, u1)
    T.tfmm_plan_store_near(plan)
    T.tfmm_evaluate(plan, M2, u2)
    T.tfmm_plan_store_near(plan, False)
    one = _held(T, plan)
    T.tfmm_evaluate(plan, M2, u2)
    assert _held(T, plan) - one >= 500 * len(tets), (_held(T, plan) - one) / len(tets)
    two = _held(T, plan)
    T.tfmm_evaluate(plan, M2, u2)
    T.tfmm_evaluate(plan, M1, u1)
    assert _held(T, plan) == two
