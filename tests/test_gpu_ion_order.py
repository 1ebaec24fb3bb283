"""The list of the ions in key order, the targets of energies and gradients: built with the cells by
one workgroup per replica up to 16,384 sources, over a grid beyond, and over a grid for a system alone
from 2,048 sources.  Whichever made it, every ion is a target once: the potentials of a replica equal
those of the same system alone, before and after a rebuild."""
import numpy as np
import pytest

from paper_1305_1825_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_1305_1825_amd import bhmc  # noqa: E402


@pytest.mark.parametrize("n,other,lines", [(1, 2, 0), (1023, 1, 0), (1024, 1025, 0), (8192, 100, 0), (8193, 100, 0),
                                           (3000, 60, 4)])
def test_every_ion_is_a_target_once(n, other, lines):
    reps = []
    for k, m in enumerate((n, other)):
        if n < 10:
            x, y, z, q = W.cube_system(m, 0, 20.0, seed=k)
            reps.append((W.make_params(p=2, box_side=20.0), x, y, z, q))
        else:
            c = W.config_colloid_10k(n=m, p=2, seed=k) if m >= 60 else None
            if c is None:
                x = np.linspace(11.0, 30.0, m)
                reps.append((reps[0][0], x, 0.0 * x, 0.0 * x, np.ones(m)))
            else:
                reps.append((dict(c["params"], line_images=lines), c["x"], c["y"], c["z"], c["q"]))
    cat = [np.concatenate([rp[k] for rp in reps]) for k in range(1, 5)]
    print("replicas of", n, other, flush=True)
    b = bhmc.Tree([rp[0] for rp in reps], *cat, n_per_replica=[n, other])
    for again in (False, True):
        for k, (P, x, y, z, q) in enumerate(reps):
            alone = bhmc.Tree(P, x, y, z, q)
            if again:
                b.rebuild(k)
                alone.rebuild()
            E, phi = alone.energy(with_phi=True)
            Eb, phib = b.energy(with_phi=True, replica=k)
            # the same groups in the same order: the same sums
            assert torch.equal(phi, phib) and E == Eb
            alone.close()
    b.close()
