"""Expansion rows as accepted moves repair them, on every path that commits moves: potentials read
from the repaired rows against those from rows summed afresh on the same tree.

A commit changes a row by at most 2 (2 + M) contributions (old and new positions of the ion, its
Kelvin image and M line images), each rounded relative to what the row holds.  By the addition
theorem the absolute products of a source's coefficients with a target's sum to at most
sum_l (d/X)^l / X <= (1 + theta) / (1 - theta) / r, so a potential drifts by at most that many times
2^-53 of sum |q| / r a move.  A contribution missing or placed in another row changes that row's
monopole by |q| and with it the potential of every ion that takes the row's cell as far by at least
|q| over the system's diameter: the tests ask for a bound far below that, and that nearly every
occupied cell is taken as far by some ion."""
import numpy as np
import pytest

from paper_1305_1825_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1305_1825_amd import bhmc  # noqa: E402


def system(n, p, **kw):
    c = W.config_colloid_10k(n=n, p=p)
    # the 10^4-ion colloid's density
    r1 = (10.5 ** 3 + n / 10000 * (40.0 ** 3 - 10.5 ** 3)) ** (1.0 / 3.0)
    x, y, z, q = W.shell_system(c["q"], 10.5, r1, 0.5, seed=n)
    return dict(W.shell_params(10.0, -50.0, 10.5, r1, hard_core=0.5, theta=0.5, p=p, leaf_cap=8), **kw), x, y, z, q


def magnitudes(P, r, q):
    """sum |q| / distance over all sources, at every ion (line images at their closest)."""
    d = np.linalg.norm(r[:, None] - r[None], axis=2)
    np.fill_diagonal(d, np.inf)
    mag = (np.abs(q)[None] / d).sum(1)
    if P["images"]:
        rn = np.linalg.norm(r, axis=1)
        img = r * (P["a"] / rn[:, None]) ** 2
        qi = np.abs(q) * P["a"] / rn
        mag += (qi[None] / np.linalg.norm(r[:, None] - img[None], axis=2)).sum(1)
        if P["line_images"]:
            mag += qi.sum() / (rn - P["a"])
    return mag


def cells_read(P, c, r):
    """Share of the occupied cells below level 1 that some ion takes through its row (N_0 = 0).  With
    line images only of those centred outside the sphere: the small cells around the centre, where the
    line images crowd, are always taken through larger ones."""
    d2 = ((r[:, None] - c["geo"][None, :, :3]) ** 2).sum(2)
    mac = 3.0 * c["geo"][:, 3] ** 2 <= P["theta"] ** 2 * d2
    reach = np.zeros_like(mac)
    reach[:, 0] = True
    for k in np.nonzero(c["link"] >= 0)[0]:  # cells are numbered level by level
        reach[:, c["link"][k]:c["link"][k] + 8] = (reach[:, k] & ~mac[:, k])[:, None]
    read = (reach & mac).any(0)
    held = (c["count"] > 0) & (c["level"] > 1)
    if P["line_images"]:
        held &= np.linalg.norm(c["geo"][:, :3], axis=1) > P["a"]
    return read[held].mean()


def check(t, P, moves, replica=0):
    x, y, z, q = (v.cpu().numpy() for v in t.state(replica))
    r = np.stack([x, y, z], 1)
    E, phi = t.energy(with_phi=True, replica=replica)
    share = cells_read(P, t.cells(replica, moments=False), r)
    t.refresh_moments(replica)
    E2, phi2 = t.energy(with_phi=True, replica=replica)
    M, th = P["line_images"], P["theta"]
    tol = 2.0 * (2 + M) * moves * 2.0 ** -53 * (1.0 + th) / (1.0 - th) * magnitudes(P, r, q)
    err = (phi - phi2).abs().cpu().numpy()
    print("moves %d: largest drift %.2g of %.2g, rows read %.3f" % (moves, err.max(), tol.max(), share), flush=True)
    assert share > 0.9
    assert tol.max() < 1e-6 / (2.0 * np.linalg.norm(r, axis=1).max())
    assert np.all(err <= tol)
    assert abs(E - E2) <= 0.5 * P["l_B"] * np.sum(np.abs(q) * tol)


@pytest.mark.parametrize("graph", [True, False])
@pytest.mark.parametrize("mpr", [0, 1])
def test_sweeps_of_replicas(graph, mpr):
    sizes = [300, 180, 424]
    reps = [W.batched_replica(k, n) for k, n in enumerate(sizes)]
    Ps = [dict(rp[0], p=5, slot_slack=1 + k) for k, rp in enumerate(reps)]  # some leaves fill up
    t = bhmc.Tree(Ps, *[np.concatenate([rp[k] for rp in reps]) for k in range(1, 5)], n_per_replica=sizes)
    t.set_moves_per_round(mpr)
    st = t.batch_sweep(seed=4, n_sweeps=100, step=1.0, use_graph=graph)
    assert sum(s["rebuilds"] for s in st) > 0 and st[2]["accepted"] > 100 * sizes[2] // 4
    for k, n in enumerate(sizes):
        check(t, Ps[k], 100 * n, replica=k)


@pytest.mark.parametrize("p,mpr,lines,slack,moves", [(0, 0, 0, 2, 400), (4, 0, 0, 1, 3000), (4, 1, 0, 1, 3000), (8, 0, 0, 2, 2000),
                                                     (10, 0, 0, 2, 400), (9, 1, 0, 2, 400), (5, 0, 2, 1, 4000), (6, 0, 8, 2, 400)])
def test_chains(p, mpr, lines, slack, moves):
    P, x, y, z, q = system(500, p, line_images=lines, slot_slack=slack)
    t = bhmc.Tree(P, x, y, z, q)
    t.set_moves_per_round(mpr)
    out = t.mc_run(seed=6, n_moves=moves, step=1.0)
    assert out["accepted"] > moves // 4
    # a rebuild sums the rows afresh; the moves since the last one are fewer than all of them
    assert slack > 1 or out["rebuilds"] > 0
    check(t, P, moves)


@pytest.mark.parametrize("p,lines", [(5, 0), (8, 0), (6, 3)])
def test_committed_moves(p, lines):
    P, x, y, z, q = system(400, p, line_images=lines, slot_slack=3)
    t = bhmc.Tree(P, x, y, z, q)
    rng = np.random.default_rng(9)
    done = 0
    for _ in range(300):
        i = int(rng.integers(len(x)))
        rn = np.array([x[i], y[i], z[i]]) + rng.random(3) - 0.5
        dE, reason = t.delta_energy(i, rn)
        if reason:
            continue
        try:
            t.commit_move(i, rn)
        except bhmc.BhmcError as e:
            assert e.code == -6  # a full leaf
            continue
        x[i], y[i], z[i] = rn
        done += 1
    assert done > 100
    check(t, P, done)
