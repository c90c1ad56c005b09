"""Infinities and NaN in one field reach every potential of that field and none
of the others'."""
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


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("form", ["fp64", "tiles", "fp32", "bf16x3", "stored", "direct"])
@pytest.mark.parametrize("F", [1, 2, 5, 9, 17])
def test_one_field_not_finite(torch_dev, F, form, value):
    import paper_1606_00247_amd as T

    torch, dev = torch_dev
    nodes, tets = meshgen.box_mesh(6 if form != "direct" else 3, seed=1)
    prec = {"fp32": T.M2L_FP32, "bf16x3": T.M2L_BF16X3}.get(form, T.M2L_FP64)
    plan = T.tfmm_plan_create(nodes, tets, p=4, leaf_size=16, theta=0.6, m2l_precision=prec)
    if form == "tiles":
        T.tfmm_plan_set_schedule(plan, 256, 0, 0, 256)
    if form == "stored":
        T.tfmm_plan_store_near(plan)
    run = T.tfmm_direct if form == "direct" else T.tfmm_evaluate
    M = meshgen.random_fields(len(nodes), F=F, seed=3)
    print("not finite", F, form, value, flush=True)
    clean = run(plan, torch.from_numpy(M).to(dev)).cpu().numpy().reshape(F, -1)
    M[F // 2, len(nodes) // 3, 1] = value
    u = run(plan, torch.from_numpy(M).to(dev)).cpu().numpy().reshape(F, -1)
    assert not np.isfinite(u[F // 2]).any()
    others = np.arange(F) != F // 2
    assert np.abs(u[others] - clean[others]).max(initial=0.0) <= 1e-13 * np.abs(clean).max()
    # nothing stays behind in the plan's buffers
    M[F // 2, len(nodes) // 3, 1] = 0.0
    u = run(plan, torch.from_numpy(M).to(dev)).cpu().numpy()
    assert np.isfinite(u).all()
