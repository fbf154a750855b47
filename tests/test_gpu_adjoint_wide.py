"""The reverse step of lattices whose adjoint populations take 4 GiB and more, which addresses each plane by
itself.  Such a lattice is 64 periods of a small one side by side: loss and gradient are means over x, so both
lattices have the same ones.  1 / lx differs by a power of two, so every site's terms do too, bit for bit,
and only the order of the FP64 sums (at most 2^28 terms) tells the results apart: relative to the largest
derivative below 1e-9, where a plane or a neighbour taken wrongly moves it by parts in a hundred."""

import numpy as np
import pytest

from cases import make_sim
from test_gpu_tile import case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lx,ly,storage,walls,bytes_per_site", [(250, 1900, "f32", True, 8), (250, 1900, "f32", False, 8),
                                                               (500, 1900, "bf16dev", True, 4)])
def test_wide_arrays(lx, ly, storage, walls, bytes_per_site):
    copies, T = 64, 3
    assert 9 * 2 * copies * lx * ly * bytes_per_site >= 1 << 32
    c = case(lx, ly, storage, 2, walls)
    c["body"] = (3e-5, 0.0)
    got = []
    for k in (1, copies):
        print(lx, ly, storage, walls, k, flush=True)
        sim = make_sim(dict(c, lx=k * lx, rho=np.tile(c["rho"], (1, 1, k))))
        got.append(sim.adjoint(T, (1.0 if walls else 0.0, 0.3), every=1, fp64_reverse=bytes_per_site == 8))
        sim.close()
    (l0, g0), (l1, g1) = got
    assert l1 == pytest.approx(l0, rel=1e-10)
    np.testing.assert_allclose(g1, g0, rtol=1e-9, atol=1e-9 * np.abs(g0[:5]).max())
