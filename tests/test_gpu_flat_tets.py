"""Near field of several fields on flat and long cells: a uniform field, whose
potential a flat tet takes from two nearly cancelling faces, against the
surface charges summed in extended precision."""
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

EPS = 2.0 ** -52
FACES = ((1, 2, 3), (0, 3, 2), (0, 1, 3), (0, 2, 1))


def _face_integrals(P, x):
    """Integrals [x] of 1/R over the triangle P [3, 3] and the sums of their terms' sizes, extended precision."""
    LD = np.longdouble
    P, x = P.astype(LD), x.astype(LD)
    n = np.cross(P[1] - P[0], P[2] - P[0])
    n = n / np.sqrt(n @ n)
    d = P[None] - x[:, None]
    R = np.sqrt((d * d).sum(axis=2))
    h = d[:, 0] @ n
    D = lambda a, b: (d[:, a] * d[:, b]).sum(axis=1)
    den = R[:, 0] * R[:, 1] * R[:, 2] + D(0, 1) * R[:, 2] + D(1, 2) * R[:, 0] + D(0, 2) * R[:, 1]
    det = (d[:, 0] * np.cross(d[:, 1], d[:, 2])).sum(axis=1)
    out = -2 * h * np.arctan2(det, den)
    size = np.abs(out)
    for p, q in ((0, 1), (1, 2), (2, 0)):
        e = P[q] - P[p]
        L = np.sqrt(e @ e)
        S = R[:, p] + R[:, q]
        edge = (d[:, p] @ np.cross(e / L, n)) * np.log((S + L) / (S - L))
        out += edge
        size += np.abs(edge)
    return out, size


def _uniform(nodes, tets, m, x):
    """(potential, sum of the terms' sizes) [x] of a uniform M: charge M.n on the
    faces that one tet has, the terms of all faces of all tets."""
    u, size = np.zeros(len(x), np.longdouble), np.zeros(len(x), np.longdouble)
    faces = {}
    for t in tets:
        v = nodes[t]
        out = 1 if np.linalg.det(v[1:] - v[0]) > 0 else -1
        for f in FACES:
            faces.setdefault(tuple(sorted(t[list(f)])), []).append((t[list(f)], out))
    for own in faces.values():
        P = nodes[own[0][0]].astype(np.longdouble)
        n = own[0][1] * np.cross(P[1] - P[0], P[2] - P[0])
        n = n / np.sqrt(n @ n)
        I, terms = _face_integrals(P, x)
        size += len(own) * np.sqrt(m @ m) * terms
        if len(own) == 1:
            u += (n @ m.astype(np.longdouble)) * I
    return u / (4 * np.pi), size / (4 * np.pi)


def _check(torch_dev, nodes, tets, x, F, seed):
    """Largest error over the sum of the terms' sizes."""
    import paper_1606_00247_amd as T

    torch, dev = torch_dev
    rng = np.random.default_rng(seed)
    m = rng.standard_normal((F, 3))
    M = np.repeat(m[:, None], len(nodes), axis=1)
    plan = T.tfmm_plan_create(nodes, tets, targets=x, theta=1e-3, leaf_size=64, p=2)
    assert T.tfmm_plan_stats(plan)["n_m2l"] == 0
    u = T.tfmm_evaluate(plan, torch.from_numpy(M).to(dev)).cpu().numpy()
    T.tfmm_plan_destroy(plan)
    worst = 0.0
    for f in range(F):
        ref, size = _uniform(nodes, tets, m[f], x)
        worst = max(worst, float((np.abs(u[f] - ref) / size).max()))
    return worst


# The closed form of a face adds its edges' terms and its solid angle's, each of
# about twenty roundings of a value and of the target's distances, up to three
# times the face's size: 64 roundings of each term.  (The same for a long face,
# whose terms cancel to a small integral.)
@pytest.mark.parametrize("F", [2, 5, 16])
@pytest.mark.parametrize("shape", [(1, 1, 0.3), (1, 1, 0.05), (1, 1, 0.003), (1, 0.001, 1), (1, 0.03, 0.001),
                                   (0.01, 1, 0.01), (1, 1, 1e-5)])
def test_one_tet(torch_dev, shape, F):
    rng = np.random.default_rng(7)
    worst = 0.0
    for turn in range(6):
        order = rng.permutation(3)
        v = np.zeros((4, 3))
        for i in range(3):
            v[i + 1] = v[i]
            v[i + 1, order[i]] += shape[order[i]]
        way = rng.standard_normal((150, 3))
        x = v.mean(axis=0) + way / np.linalg.norm(way, axis=1)[:, None] * rng.uniform(1.0, 3.0, (150, 1))
        print("flat tet", shape, F, turn, flush=True)
        worst = max(worst, _check(torch_dev, v, np.array([[0, 1, 2, 3]], np.int32), x, F, turn))
    assert worst <= 64 * EPS, worst / EPS


@pytest.mark.parametrize("h", [0.1, 0.01, 0.003])
def test_flat_cells(torch_dev, h):
    nodes, tets = meshgen.box_mesh((4, 3, 2), seed=1)
    lo, hi = nodes.min(axis=0), nodes.max(axis=0)
    nodes = (nodes - lo) / (hi - lo) * np.array([4, 3, 2 * h])
    rng = np.random.default_rng(2)
    x = np.array([-3, -3, 0]) + np.array([10, 9, 0]) * rng.random((200, 3))
    x[:, 2] = rng.choice([-1.0, 1.0], 200) * rng.uniform(1.0, 3.0, 200)
    print("flat cells", h, flush=True)
    worst = _check(torch_dev, nodes, tets, x, 3, 5)
    assert worst <= 64 * EPS, worst / EPS
