"""Near leaves around the sizes at which their slots are found another way, from a list of every
slot's leaf or by search: more than 64 slots an entry on average, or more than the list holds.  A
system in one leaf has every source in one near entry a move (64 ions and 65); leaves of a split
system with many, few and no members, on both sides of the average and of the list's capacity
(2,048 slots one move at a time, 4,096 in rounds)."""
import numpy as np
import pytest

import oracle as O
from paper_1305_1825_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1305_1825_amd import bhmc  # noqa: E402

CASES = [(2, 5000), (64, 5000), (65, 5000), (513, 5000), (2049, 5000), (1500, 400), (1500, 33), (3000, 60), (3000, 64),
         (3000, 70), (6000, 60)]


def system(n, leaf):
    side = 20.0 * (n / 1000.0) ** (1.0 / 3.0)
    x, y, z, q = W.cube_system(n - n // 2, n // 2, side, seed=n)
    if leaf < 5000:  # a dense corner beside sparse cells
        k = n // 3
        x[:k] *= 0.2; y[:k] *= 0.2; z[:k] *= 0.2
    return W.make_params(theta=0.4, p=2, leaf_cap=leaf, box_side=side, slot_slack=3), x, y, z, q


@pytest.mark.parametrize("n,leaf", CASES)
@pytest.mark.parametrize("rounds", [0, 1])
def test_moves_over_leaves_of_every_size(n, leaf, rounds):
    P, x, y, z, q = system(n, leaf)
    g = bhmc.Tree(P, x, y, z, q)
    g.set_moves_per_round(rounds)
    o = O.Tree(P, x, y, z, q)
    print("n=%d leaf=%d rounds=%d cells=%d" % (n, leaf, rounds, g.info()["ncell"]), flush=True)
    r = np.stack([x, y, z], 1)
    for m in range(4):
        i, d, _ = O.draw_move(11, 0, m, n, 0.5)
        rn = r[i] + d
        dE, reason = g.delta_energy(i, rn)
        dEo, ro = o.delta(i, rn)
        assert reason == ro
        if not ro:
            mag = sum(np.sum(np.abs(q)[np.arange(n) != i] / np.linalg.norm((r - at)[np.arange(n) != i], axis=1))
                      for at in (r[i], rn))
            assert abs(dE - dEo) <= 1e-12 * P["l_B"] * abs(q[i]) * mag
    moves = 60
    a = g.mc_run(seed=5, n_moves=moves, step=0.5, accept_bits=True)["accept"].cpu().numpy()
    assert np.array_equal(a, o.mc_run(seed=5, replica=0, move0=0, n_moves=moves, step=0.5)["accept"])
    xo, yo, zo, _ = o.sources()
    for u, v in zip(g.state(), (xo, yo, zo)):
        assert np.array_equal(u.cpu().numpy(), v)
    g.close()
