"""Frontiers of rounds of trial moves at theta = 0, where a level holds an entry for every cell
and every move of the round: the widest a traversal's frontier gets.  The cell counts are such
that the widest level holds most of the tree's cells, so a level of a round has more than four
times as many entries as the tree has cells."""
import numpy as np
import pytest

import oracle as O
from paper_1305_1825_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1305_1825_amd import bhmc  # noqa: E402


def cube(n, seed):
    side = 20.0 * (n / 1000.0) ** (1.0 / 3.0)
    x, y, z, q = W.cube_system(n // 2, n - n // 2, side, seed=seed)
    return W.make_params(theta=0.0, p=1, leaf_cap=16, box_side=side), x, y, z, q


def widest(g):
    lev = g.cells(moments=False)["level"]
    return int(np.bincount(lev).max()), len(lev)


@pytest.mark.parametrize("p", [1, 9])
def test_theta_zero_chain_in_rounds_equals_oracle(p):
    P, x, y, z, q = cube(20000, 1)
    P = dict(P, p=p)
    g = bhmc.Tree(P, x, y, z, q)
    width, ncell = widest(g)
    print("theta=0 rounds: n=20000 p=%d cells=%d widest level=%d" % (p, ncell, width), flush=True)
    assert 8 * width > 4 * ncell
    r = g.mc_run(seed=3, n_moves=24, step=1.0, accept_bits=True)
    o = O.Tree(P, x, y, z, q)
    ro = o.mc_run(seed=3, replica=0, move0=0, n_moves=24, step=1.0)
    assert np.array_equal(r["accept"].cpu().numpy(), ro["accept"])
    xs, ys, zs, _ = (t.cpu().numpy() for t in g.state())
    xo, yo, zo, _ = o.sources()
    assert np.array_equal(xs, xo) and np.array_equal(ys, yo) and np.array_equal(zs, zo)
    # the handle's other traversals on the same regions: each potential sums n terms of at least
    # 1 / (sqrt(3) side), a few roundings each
    phi = g.energy(with_phi=True)[1].cpu().numpy()
    phio = o.energy(with_phi=True)[1]
    assert np.all(np.abs(phi - phio) <= 1e-12 * len(x) / (3.0 ** 0.5 * P["box_side"]))
    g.close()


def test_theta_zero_replicas_in_rounds_equal_oracle():
    sizes = [9000, 300]
    reps = [cube(n, k) for k, n in enumerate(sizes)]
    cat = [np.concatenate([rp[k] for rp in reps]) for k in range(1, 5)]
    g = bhmc.Tree([rp[0] for rp in reps], *cat, n_per_replica=sizes)
    print("theta=0 rounds: replicas of", sizes, flush=True)
    st = g.batch_sweep(seed=2, n_sweeps=1, step=1.0)
    for k, (P, x, y, z, q) in enumerate(reps):
        o = O.Tree(P, x, y, z, q)
        ro = o.mc_run(seed=2, replica=k, move0=0, n_moves=sizes[k], step=1.0)
        assert st[k]["accepted"] == ro["stats"][0]
        xs, ys, zs, _ = (t.cpu().numpy() for t in g.state(k))
        xo, yo, zo, _ = o.sources()
        assert np.array_equal(xs, xo) and np.array_equal(ys, yo) and np.array_equal(zs, zo)
    g.close()
