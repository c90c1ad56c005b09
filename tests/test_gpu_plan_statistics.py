"""The plan's statistics count all the device memory that it holds."""
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


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16x6"])
@pytest.mark.parametrize("F", [1, 5, 16])
def test_statistics_count_what_is_held(torch_dev, F, precision):
    import paper_1606_00247_amd as T

    torch, dev = torch_dev
    prec = {"fp64": T.M2L_FP64, "fp32": T.M2L_FP32, "bf16x6": T.M2L_BF16X6}[precision]
    used = {}
    for n in (3, 26):  # the small one first: what the runtime allocates once
        nodes, tets = meshgen.box_mesh(n, seed=1)
        M, u = _fields(torch_dev, len(nodes), F)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        plan = T.tfmm_plan_create(nodes, tets, p=8, leaf_size=32, theta=0.5, m2l_precision=prec)
        T.tfmm_evaluate(plan, M, u)
        torch.cuda.synchronize()
        used[n] = (free - torch.cuda.mem_get_info()[0], _held(T, plan))
        T.tfmm_plan_destroy(plan)
    real, said = used[26]
    # about sixty allocations, each rounded up to at most 2 MiB
    print("memory", F, precision, real, said, flush=True)
    assert said <= real <= said + (120 << 20), (real / 2**20, said / 2**20)
    assert said >= 0.8 * real
