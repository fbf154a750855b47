"""The passes over the current state (moments, totals, profile, stress field) at the edges of their tiles
(64 x 8 sites; 16 x 8 where those are fewer than the compute units and nothing is summed): narrower than
a tile's frame, one more and one less than a tile, ragged, and large enough for the wide tile.  FP64
against the oracle on the same state: fields and sums of at most 2^18 terms agree to 1e-10 of the largest
value (rounding 1e-16; velocities and sums are differences of terms up to 1e5 times larger)."""

import numpy as np
import pytest

from cases import make_oracle, make_sim
from test_gpu_tile import case

pytestmark = pytest.mark.gpu


def near(got, ref):
    ref = np.asarray(ref)
    np.testing.assert_allclose(np.asarray(got), ref, rtol=1e-10, atol=1e-10 * max(np.abs(ref).max(), 1e-300))


@pytest.mark.parametrize("lx,ly", [(5, 5), (15, 9), (63, 17), (65, 8), (257, 70), (1030, 129)])
@pytest.mark.parametrize("ns,walls", [(1, False), (2, True), (2, False)])
def test_passes_at_tile_edges(lx, ly, ns, walls):
    import torch
    from oracle import diagnostics as dg
    c = case(lx, ly, "f64", ns, walls)
    c["body"] = (3e-5, 1e-5)  # sums that do not vanish
    sim, orc = make_sim(c), make_oracle(c)
    sim.step(3)
    orc.step(3)
    fl = orc.fields()
    print(lx, ly, ns, walls, flush=True)
    rho, u = (t.cpu().numpy() for t in sim.moments())
    near(rho, fl["rho"])
    near(u, fl["u"])
    assert np.array_equal(sim.moments(dtype=torch.float32)[0].cpu().numpy(), rho.astype(np.float32))
    near(sim.stress_field().cpu().numpy(), np.stack(dg.stress_field(orc)))
    m, p, q = sim.totals()
    near(m[:ns], fl["rho"].sum(axis=(1, 2)))
    near(p, fl["j"].sum(axis=(0, 2, 3)))
    near(q, fl["u"][0].sum() / lx)
    prof = sim.profile().cpu().numpy()
    ubar, sigma = dg.shear_profile(orc)
    near(prof[:ly], ubar)
    # a line's stress: differences of populations and pair forces of the order of the density, rounded
    # to 1e-16 each, whatever is left of them (1e-7 in the nearly uniform film)
    assert np.abs(prof[ly:2 * ly + 1] - sigma).max() <= 1e-14 * fl["rho"].max()
    near(prof[2 * ly + 1:3 * ly + 1], fl["rho"][0].mean(axis=1))
    sim.close()
