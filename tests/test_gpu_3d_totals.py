"""The totals of a three-dimensional lattice do not depend on the kernel that steps it: the momentum of a
periodic lattice near rest is what rounding leaves of a sum that cancels (1e-13 of a sum of |j| of 1e4 or
more), so its digits are those of the order of the additions.  The default context and one whose launch
shape was set to the very shape the default reports have to give the same numbers, bit for bit."""

import numpy as np
import pytest

import lbgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lx,ly,lz", [(37, 9, 6), (64, 48, 40), (96, 60, 56), (65, 49, 130)])
@pytest.mark.parametrize("storage,ns,walls", [("f64", 2, False), ("f64", 1, False), ("f32", 2, False), ("f64", 2, True)])
def test_totals_are_those_of_the_set_shape(lx, ly, lz, storage, ns, walls):
    from paper_1402_6019_amd import Sim3
    rich = np.random.default_rng(lx).uniform(0.0, 1.0, (lz, ly, lx)) < 0.6
    rho = np.stack([np.where(rich, 1.2, 0.2), np.where(rich, 0.2, 1.2)])[:ns]
    kw = dict(n_species=ns, walls=walls, storage=storage, g1=lbgen.EMULSION_G1, g2=lbgen.EMULSION_G2,
              gab=lbgen.EMULSION_GAB, rho0=lbgen.EMULSION_RHO0, rho_ref=(0.7, 0.7))
    if walls:
        kw.update(body=(1e-6, 0.0, 0.0), rho_wall=lbgen.EMULSION_POOR)
    print(lx, ly, lz, storage, ns, walls, flush=True)
    got = []
    for shape in (False, True):
        sim = Sim3(lx, ly, lz, rho, **kw)
        if shape:
            sim.set_tile(*sim.get_tile())
        sim.step(7)
        m, p, q = sim.totals()
        got.append([*m, *p, q])
        sim.close()
    assert got[0] == got[1]
