"""More leaves times fields than one launch of the multipole kernel can hold
(2^32 threads in a direction of the grid)."""
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


def test_leaves_times_fields(torch_dev):
    import paper_1606_00247_amd as T

    torch, dev = torch_dev
    nodes, tets = meshgen.box_mesh(11, seed=1)
    plan = T.tfmm_plan_create(nodes, tets, p=1, leaf_size=1, theta=0.5)
    cells, _ = T.tfmm_plan_cells(plan)
    parents = {(c[0] - 1, c[1] >> 1, c[2] >> 1, c[3] >> 1) for c in cells}
    leaves = sum(1 for c in cells if c[4] > 0 and tuple(c[:4]) not in parents)
    F = 10000
    print("many fields", leaves, F, flush=True)
    assert leaves * (F // 4) * 256 > 2 ** 32
    g = torch.Generator(device=dev).manual_seed(1)
    M = torch.randn((F, len(nodes), 3), dtype=torch.float64, device=dev, generator=g)
    u = T.tfmm_evaluate(plan, M)
    for f in (0, 1, F // 2, F - 2, F - 1):
        one = T.tfmm_evaluate(plan, M[f].contiguous())
        assert float((u[f] - one).abs().max()) <= 1e-12 * float(one.abs().max()), f
