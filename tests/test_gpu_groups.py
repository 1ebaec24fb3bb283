"""Energies, gradients and builds of whole systems at the edges of their grid-wide forms: fewer ions than a group,
one more or less than a multiple, the sizes at which the group grows, the N_0 rule, systems
without images, the single-precision far field, and frontiers that leave the chip."""
import numpy as np
import pytest

import oracle as O
from paper_1305_1825_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1305_1825_amd import bhmc  # noqa: E402

CASES = [  # system, ions, order, theta, N_0, frontier entries on chip
    ("colloid", 60, 5, 0.5, 0, 4096), ("colloid", 63, 4, 0.5, 3, 4096), ("colloid", 65, 0, 0.5, 0, 64),
    ("cube", 1, 4, 0.5, 0, 4096), ("cube", 2, 4, 0.5, 0, 4096), ("cube", 5, 3, 0.9, 1, 4096),
    ("cube", 17, 10, 0.7, 0, 4096), ("cube", 4095, 3, 0.5, 0, 4096), ("cube", 4097, 3, 0.5, 8, 64),
    ("colloid", 4099, 6, 0.3, 0, 64), ("cube", 16383, 2, 0.6, 0, 4096), ("cube", 16387, 2, 0.6, 0, 4096),
    ("colloid", 777, 8, 0.0, 0, 4096), ("cube", 2048, 3, 0.5, 0, 4096), ("cube", 2049, 3, 0.5, 0, 4096),
]


def system(kind, n, p, theta, n0):
    if kind == "cube":
        side = 20.0 * (max(n, 8) / 1000.0) ** (1.0 / 3.0)
        x, y, z, q = W.cube_system(n - n // 2, n // 2, side, seed=n)
        return W.make_params(theta=theta, p=p, leaf_cap=8, box_side=side, n0=n0), x, y, z, q
    c = W.config_colloid_10k(n=n, p=p, theta=theta)
    return dict(c["params"], n0=n0), c["x"], c["y"], c["z"], c["q"]


@pytest.mark.parametrize("kind,n,p,theta,n0,front", CASES)
def test_energy_and_potentials_match_oracle(kind, n, p, theta, n0, front):
    P, x, y, z, q = system(kind, n, p, theta, n0)
    g = bhmc.Tree(P, x, y, z, q)
    g.set_frontier_capacity(front)
    print(kind, n, p, theta, n0, front, flush=True)
    E, phi = g.energy(with_phi=True)
    Eo, phio = O.Tree(P, x, y, z, q).energy(with_phi=True)
    phi = phi.cpu().numpy()
    # a potential's sum of at most 2 n terms, each a few roundings off: 1e-12 of its terms' sum,
    # bounded by that of |q| / distance (images included)
    r = np.stack([x, y, z], 1)
    mag = np.full(n, 1e-300)
    for i in range(0, n, 512):
        d = np.linalg.norm(r[i:i + 512, None] - r[None], axis=2)
        d[np.arange(d.shape[0]), np.arange(i, i + d.shape[0])] = np.inf
        mag[i:i + 512] += (np.abs(q)[None] / d).sum(1)
    mag = 2.0 * mag + 2.0
    assert np.all(np.abs(phi - phio) <= 1e-12 * mag), np.max(np.abs(phi - phio) / mag)
    assert abs(E - Eo) <= 1e-12 * np.sum(np.abs(q) * mag)


@pytest.mark.parametrize("n", [61, 2048, 2049, 4100])
def test_single_precision_far_field_excludes_the_own_image_exactly(n):
    """Where every far cell but the one with the own image is replaced by its single-precision
    value, the potential stays within that rounding of the FP64 one."""
    P, x, y, z, q = system("colloid", n, 4, 0.5, 0)
    _, phi = bhmc.Tree(P, x, y, z, q).energy(with_phi=True)
    _, phi32 = bhmc.Tree(dict(P, far_fp32=1), x, y, z, q).energy(with_phi=True)
    o = O.Tree(P, x, y, z, q)
    K = (35 + 3 * 4 + 4) * 2.0 ** -24
    for i in range(0, n, max(1, n // 40)):
        mag = o.far_magnitude(np.array([x[i], y[i], z[i]]), (i, n + i))
        assert abs(float(phi[i] - phi32[i])) <= K * mag + 1e-12 * (1.0 + abs(float(phi[i])))


GRAD_CASES = [  # system, ions, order, theta, N_0, frontier entries on chip, leaf capacity
    ("cube", 1, 4, 0.5, 0, 4096, 8), ("cube", 2, 5, 0.5, 0, 4096, 8), ("cube", 15, 6, 0.9, 0, 4096, 2),
    ("cube", 33, 1, 0.7, 2, 4096, 1), ("colloid", 63, 0, 0.5, 0, 64, 8), ("colloid", 80, 7, 0.6, 0, 4096, 4),
    ("colloid", 401, 9, 0.5, 0, 4096, 1), ("colloid", 257, 10, 0.5, 4, 64, 8), ("colloid", 1025, 3, 0.3, 0, 64, 8),
]


@pytest.mark.parametrize("kind,n,p,theta,n0,front,leaf", GRAD_CASES)
def test_gradient_matches_oracle(kind, n, p, theta, n0, front, leaf):
    P, x, y, z, q = system(kind, n, p, theta, n0)
    P = dict(P, leaf_cap=leaf)
    g = bhmc.Tree(P, x, y, z, q)
    g.set_frontier_capacity(front)
    print(kind, n, p, theta, n0, front, flush=True)
    E, dr, dq = g.energy_grad()
    o = O.Tree(P, x, y, z, q)
    Eo = o.energy()
    go, gqo = o.grad()[-2:]
    dr, dq = dr.cpu().numpy(), dq.cpu().numpy()
    go = np.asarray(go).reshape(n, 3)
    rms = np.sqrt(np.mean(go ** 2)) + 1e-300
    assert np.all(np.abs(dr - go) <= 1e-10 * (np.abs(go) + rms)), np.max(np.abs(dr - go) / (np.abs(go) + rms))
    assert np.all(np.abs(dq - gqo) <= 1e-10 * (np.abs(gqo) + 1.0))
    assert abs(E - Eo) <= 1e-11 * max(1.0, np.sum(np.abs(q) * np.abs(gqo)))


def test_gradient_after_moves_with_a_single_precision_far_field():
    """Its moves repair the moments the single-precision copy is made of; the gradient, always
    in FP64, forms its expansion rows from them."""
    P, x, y, z, q = system("colloid", 400, 5, 0.5, 0)
    t = bhmc.Tree(dict(P, far_fp32=1), x, y, z, q)
    t.mc_run(seed=3, n_moves=200, step=1.0)
    E, dr, dq = t.energy_grad()
    t.refresh_moments()
    E2, dr2, dq2 = t.energy_grad()
    s = float(dr2.abs().max())
    assert float((dr - dr2).abs().max()) <= 1e-11 * s and float((dq - dq2).abs().max()) <= 1e-11 * float(dq2.abs().max())
    xs, ys, zs, qs = (v.cpu().numpy() for v in t.state())
    f = bhmc.Tree(P, xs, ys, zs, qs)
    assert abs(E - E2) <= 1e-11 * max(1.0, abs(E2))
    # a fresh FP64 tree of the same ions has the cells of the current positions, not of the built
    # ones: its gradient differs by truncation only (order 5 at theta = 0.5)
    _, dr3, _ = f.energy_grad()
    assert float((dr2 - dr3).abs().max()) <= 1e-2 * s


@pytest.mark.parametrize("n,leaf,depth", [(1024, 16, 21), (1025, 1, 21), (1500, 0, 5), (4100, 200000, 21), (2500, 3, 0),
                                          (2500, 3, 1), (20001, 16, 21)])
def test_grid_build_equals_the_one_workgroup_build(n, leaf, depth):
    """Sizes from which a single replica's tree is built over a grid (2,048 sources), one-source
    leaves, uniform trees, and trees of one cell or one level, against the same replica in a handle
    of two, built by one workgroup."""
    c = W.config_colloid_10k(n=n, p=4)
    P = dict(c["params"], leaf_cap=leaf, max_depth=depth)
    print(n, leaf, depth, flush=True)
    a = bhmc.Tree(P, c["x"], c["y"], c["z"], c["q"])
    two = [np.concatenate([c[k], c[k][:100]]) for k in "xyzq"]
    b = bhmc.Tree([P, P], *two, n_per_replica=[n, 100])
    assert a.info() == b.info(0)
    for u, v in zip(a.sorted(), b.sorted(0)):
        assert np.array_equal(u, v)
    ca, cb, la, lb = a.cells(), b.cells(0), a.leaves(), b.leaves(0)
    assert all(np.array_equal(ca[k], cb[k]) for k in ca) and all(np.array_equal(la[k], lb[k]) for k in la)
    assert all(np.array_equal(u, v) for u, v in zip(a.leaf_members(), b.leaf_members(0)))
    assert a.energy() == b.energy()
