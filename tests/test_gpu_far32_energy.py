"""Potentials with the single-precision far field at the sizes and orders at which the groups of the
energy traversal change, within the rounding bound K 2^-24 sum |T_n M^n| of a far cell's
single-precision value, K = C(p+3,3) + 3p + 4."""
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


@pytest.mark.parametrize("p,n", [(2, 4096), (2, 4097), (4, 4096), (4, 4097), (5, 3072), (5, 3073), (6, 2048), (6, 2049)])
def test_potentials(p, n):
    P, x, y, z, q = system(n, p)
    _, phi = bhmc.Tree(P, x, y, z, q).energy(with_phi=True)
    _, phi32 = bhmc.Tree(dict(P, far_fp32=1), x, y, z, q).energy(with_phi=True)
    o = O.Tree(P, x, y, z, q)
    d = (phi - phi32).abs().cpu().numpy()
    scale = float(phi.abs().max())
    for i in range(0, n, n // 40):
        mag = o.far_magnitude(np.array([x[i], y[i], z[i]]), (i, n + i))
        assert d[i] <= k_of(p) * EPS32 * mag + 1e-12 * scale
