"""Far rules of the direct sum at their distances: single tets, every nodal
field at once (the error is linear in the nodal M, so its largest value over
|M_i| <= 1 is the sum over the corners of the error vectors' lengths), targets
along the edges, where a long tet is integrated worst."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    return torch, torch.device("cuda:0")

# from (longest edges), points in a direction, error there relative to
# |M| V / (4 pi d^2); it falls as distance^(-2 n)
RULES = ((3.0, 7, 7.0e-14), (6.0, 6, 2.2e-15), (12.0, 5, 1.7e-15), (24.0, 4, 2.3e-14))
# twelve components of about a dozen roundings each, of a quarter of the whole
ROUNDING = 32 * 2.0 ** -52

SHAPES = {
    "regular": [[1, 1, 1], [1, -1, -1], [-1, 1, -1], [-1, -1, 1]],
    "kuhn": [[0, 0, 0], [1, 0, 0], [1, 1, 0], [1, 1, 1]],
    # corners in the orders that these are worst in
    "needle": [[0, 0, 0], [0, 0, 1], [0.001, 0, 0], [0, 0.001, 0]],
    "needle from a corner": [[1, 0, 0], [0, 0, 0], [1, 0, 0.001], [1, 0.001, 0]],
    "flat": [[0, 0, 0], [1, 0, 0], [0.5, 0.5, 0.02], [0.5, -0.5, 0.02]],
}


def _reference(v, x, n=20):
    """Potentials [x, corner, axis] of the unit nodal fields by a collapsed Gauss rule in extended precision."""
    t, w = np.polynomial.legendre.leggauss(n)
    t, w = (t.astype(np.longdouble) + 1) / 2, w.astype(np.longdouble) / 2
    a, b, c = (q.ravel() for q in np.meshgrid(t, t, t, indexing="ij"))
    wa, wb, wc = (q.ravel() for q in np.meshgrid(w, w, w, indexing="ij"))
    lam = np.stack([np.zeros_like(a), a, b * (1 - a), c * (1 - a) * (1 - b)], axis=1)
    lam[:, 0] = 1 - lam.sum(axis=1)
    v = v.astype(np.longdouble)
    vol6 = abs(np.dot(v[1] - v[0], np.cross(v[2] - v[0], v[3] - v[0])))
    d = x.astype(np.longdouble)[:, None] - (lam @ v)[None]
    r2 = (d * d).sum(axis=2)
    g = (wa * wb * wc * (1 - a) ** 2 * (1 - b) * vol6)[None] / (r2 * np.sqrt(r2))
    return np.stack([((g * lam[:, i])[:, :, None] * d).sum(axis=1) for i in range(4)], axis=1) / (4 * np.pi)


@pytest.mark.parametrize("shape", sorted(SHAPES))
def test_far_rule_error_over_all_fields(torch_dev, shape):
    import paper_1606_00247_amd as T

    torch, dev = torch_dev
    v = np.array(SHAPES[shape], float)
    c = v.mean(axis=0)
    pairs = [(i, j) for i in range(4) for j in range(i)]
    size = max(np.linalg.norm(v[i] - v[j]) for i, j in pairs)
    ways = [v[i] - v[j] for i, j in pairs]
    ways = [s * q / np.linalg.norm(q) for q in ways for s in (1.0, -1.0)]
    ratios = [3.001, 4.0, 5.001, 5.999, 6.001, 9.001, 11.999, 12.001, 18.0, 23.999, 24.001, 60.0]
    at = np.repeat(ratios, len(ways))
    x = c + size * at[:, None] * np.tile(ways, (len(ratios), 1))
    ref = _reference(v, x)
    M = np.eye(12).reshape(12, 4, 3)
    plan = T.tfmm_plan_create(v, np.array([[0, 1, 2, 3]], np.int32), targets=x, p=2, leaf_size=4, theta=0.5)
    vol = abs(np.linalg.det(v[1:] - v[0])) / 6
    d2 = ((x - c) ** 2).sum(axis=1)
    r, n, e = np.array(RULES)[np.searchsorted([q[0] for q in RULES], at) - 1].T
    allowed = (1.05 * e * (r / at) ** (2 * n) + ROUNDING) * vol / (4 * np.pi * d2)
    for F in (1, 12):
        print("far rules", shape, F, flush=True)
        u = np.concatenate([T.tfmm_direct(plan, torch.from_numpy(M[f:f + F]).to(dev)).cpu().numpy().reshape(F, -1)
                            for f in range(0, 12, F)])
        err = u.T.reshape(-1, 4, 3) - ref
        worst = np.sqrt((err * err).sum(axis=2)).sum(axis=1).astype(float)
        bad = worst > allowed
        assert not bad.any(), (F, at[bad], (worst / (vol / (4 * np.pi * d2)))[bad])
