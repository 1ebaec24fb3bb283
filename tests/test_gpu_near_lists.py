"""Near leaves around the sizes at which their slots are listed another way: by one lane, by the
entry's wave, or (more slots than the list holds) found by search.  A system in one leaf has every
source in one near entry a move: 32 slots and 33; 512 ions and 513 in rounds of eight moves, 2,048
and 2,049 one move at a time for the list's capacity.  Leaves of a split system with many, few and
no members between."""
import numpy as np
import pytest

import oracle as O
from paper_1305_1825_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1305_1825_amd import bhmc  # noqa: E402

CASES = [(31, 5000), (32, 5000), (33, 5000), (65, 5000), (512, 5000), (513, 5000), (2048, 5000), (2049, 5000),
         (1500, 400), (1500, 33), (3000, 700)]


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
