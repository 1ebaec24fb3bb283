"""The single-precision far field of moves on both sides of the order from which a lane takes one
target of a move instead of both (5; in 256-thread workgroups 8, in their rounds 9), within the rounding
bound K 2^-24 sum |T_n M^n| of a far cell's single-precision value, K = C(p+3,3) + 3p + 4."""
import math

import numpy as np
import pytest

import oracle as O
from paper_1305_1825_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1305_1825_amd import bhmc  # noqa: E402

EPS32 = 2.0 ** -24


def k_of(p):
    return O.nterms(p) + 3 * p + 4


def system(n, p, **kw):
    c = W.config_colloid_10k(n=n, p=p)
    return dict(c["params"], **kw), c["x"], c["y"], c["z"], c["q"]


@pytest.mark.parametrize("p,n0,lines", [(0, 0, 0), (4, 0, 0), (5, 0, 0), (5, 6, 0), (6, 0, 2), (9, 0, 0), (10, 0, 0)])
def test_energy_changes(p, n0, lines):
    P, x, y, z, q = system(600, p, n0=n0, line_images=lines, leaf_cap=8)
    n = len(x)
    f = bhmc.Tree(dict(P, far_fp32=1), x, y, z, q)
    g = bhmc.Tree(P, x, y, z, q)
    o = O.Tree(P, x, y, z, q)
    print("p=%d n0=%d lines=%d" % (p, n0, lines), flush=True)
    for m in range(30):
        i, d, _ = O.draw_move(5, 0, m, n, 1.0)
        at = np.array([x[i], y[i], z[i]])
        dE, reason = g.delta_energy(i, at + d)
        dF, reason_f = f.delta_energy(i, at + d)
        assert reason == reason_f
        if reason:
            continue
        # the mover's line images stay in the traversal's far cells
        ex = [i, n + i]
        bound = k_of(p) * EPS32 * P["l_B"] * abs(q[i]) * (o.far_magnitude(at + d, ex) + o.far_magnitude(at, ex))
        scale = max(abs(dE), P["l_B"] * abs(q[i]) * abs(o.phi(at, ex)))
        assert abs(dE - dF) <= bound + 1e-11 * scale, (m, dE, dF, bound)


@pytest.mark.parametrize("p", [4, 5, 10])
@pytest.mark.parametrize("rounds", [0, 1])
def test_chains(p, rounds):
    check_chain(p, rounds, 0)


@pytest.mark.parametrize("p,rounds", [(5, 0), (8, 0), (9, 0), (7, 1), (8, 1)])
def test_256_threads(p, rounds):
    """There a lane takes one target from order 9 on in rounds, from 8 on one move at a time."""
    check_chain(p, rounds, 1)


def check_chain(p, rounds, shape):
    P, x, y, z, q = system(500, p)
    n, moves = len(x), 300
    g = bhmc.Tree(dict(P, far_fp32=1), x, y, z, q)
    g.set_shape(shape)
    g.set_moves_per_round(rounds)
    print("p=%d rounds=%d shape=%d" % (p, rounds, shape), flush=True)
    bits = g.mc_run(seed=1, n_moves=moves, step=1.0, accept_bits=True)["accept"].cpu().numpy()
    o = O.Tree(P, x, y, z, q)
    ro = o.mc_run(seed=1, replica=0, move0=0, n_moves=moves, step=1.0)
    first = np.nonzero(bits != ro["accept"])[0]
    if len(first) == 0:
        xo, yo, zo, _ = o.sources()
        for u, v in zip(g.state(), (xo, yo, zo)):
            assert np.array_equal(u.cpu().numpy(), v[:n])
        return
    # the chains may part only where the Metropolis margin is within the bound
    k = int(first[0])
    o2 = O.Tree(P, x, y, z, q)
    o2.mc_run(seed=1, replica=0, move0=0, n_moves=k, step=1.0)
    xo, yo, zo, _ = o2.sources()
    i, d, al = O.draw_move(1, 0, k, n, 1.0)
    at = np.array([xo[i], yo[i], zo[i]])
    bound = k_of(p) * EPS32 * P["l_B"] * abs(q[i]) * (o2.far_magnitude(at + d, [i, n + i]) + o2.far_magnitude(at, [i, n + i]))
    assert abs(math.log(al) + ro["dE"][k]) <= bound + 1e-9
