"""The default 3-D step kernels (the march with its register FIFO, and the split step of small
lattices) against the kernel of a set launch shape, which the oracle tests pin: the per-site
arithmetic is the same expressions in the same order, so populations and moments agree bit for bit;
totals are FP64 sums in another order (relative 1e-12 of sums of at most 1e6 positive terms, the
momentum relative to the mass)."""

import numpy as np
import pytest

import lbgen

pytestmark = pytest.mark.gpu

# split: a lattice narrower than a tile and its frames, one with ragged tiles on every axis; march
# (segments of more than eight planes): ragged, whole tiles, and FP64's smaller tiles
SIZES = [(5, 5, 5), (37, 9, 6), (70, 21, 13), (65, 49, 130), (290, 131, 34)]


@pytest.mark.parametrize("lx,ly,lz", SIZES)
@pytest.mark.parametrize("storage,ns,walls,cross", [("f64", 2, True, False), ("f64", 1, False, False), ("f32", 2, False, True),
                                                    ("f32", 2, True, False), ("f32", 1, True, False)])
def test_default_3d_step_is_bitwise_the_set_shape(lx, ly, lz, storage, ns, walls, cross):
    from paper_1402_6019_amd import Sim3
    a = np.random.default_rng(lx + ly).uniform(0.3, 1.1, (lz, ly, lx))
    rho = np.stack([a, 1.4 - a])[:ns]
    kw = dict(n_species=ns, walls=walls, storage=storage, g1=lbgen.EMULSION_G1, g2=lbgen.EMULSION_G2,
              gab=lbgen.EMULSION_GAB, rho0=lbgen.EMULSION_RHO0, tau=(0.9, 1.2), cross_psi=cross, rho_ref=(0.7, 0.7))
    if walls:
        kw.update(body=(1e-5, 0.0, 2e-5), rho_wall=lbgen.EMULSION_POOR)
    print(lx, ly, lz, storage, ns, walls, cross, flush=True)
    out = []
    for tile in (None, (4, 16)):
        sim = Sim3(lx, ly, lz, rho, tile=tile, **kw)
        sim.step(4)
        m, p, q = sim.totals()
        r, u = sim.moments()
        sim.step(1)
        out.append((sim.checkpoint().cpu().numpy(), r.cpu().numpy(), u.cpu().numpy(), np.array([*m, *p, q])))
        sim.close()
    for x, y in zip(out[0][:3], out[1][:3]):
        assert np.array_equal(x, y)
    mass = out[1][3][0] + out[1][3][1]
    assert np.abs(out[0][3][:5] - out[1][3][:5]).max() <= 1e-12 * mass
    assert abs(out[0][3][5] - out[1][3][5]) <= 1e-12 * mass  # sum u_x / (lx lz), |u| < 1
