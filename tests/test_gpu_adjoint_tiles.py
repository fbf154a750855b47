"""The reverse step's tiles (16 x 8, 16 x 16, 32 x 16 sites, by the number of tiles) at ragged edges and on
lattices narrower than a tile's neighbourhood, against the oracle's complex-step gradient.  Each
derivative sums steps x sites terms (at most 2^20) in FP64: relative to the largest one, rounding and
cancellation stay below 1e-9; a wrong frame site moves it by about one part in the number of sites."""

import numpy as np
import pytest

from cases import make_oracle, make_sim, oracle_params
from test_gpu_tile import case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lx,ly", [(7, 5), (17, 9), (61, 37), (241, 262), (517, 270)])
@pytest.mark.parametrize("ns,walls", [(1, False), (2, True), (2, False)])
def test_reverse_tiles_match_the_complex_step(lx, ly, ns, walls):
    from oracle import cs_grad
    c = case(lx, ly, "f64", ns, walls)
    c["body"] = (3e-5, 0.0)
    T, lw = 5, (1.0 if walls else 0.0, 0.3)
    sim = make_sim(c)
    loss, g7 = sim.adjoint(T, lw, every=3)
    sim.close()
    P, f0 = oracle_params(c), make_oracle(c).get_f()
    ref = [cs_grad(P, f0, T, lw, k) for k in range(4)]
    d = np.array([r[1] for r in ref])
    got = np.array([g7[0] + g7[1], g7[2] + g7[3], g7[4], g7[5]])
    assert loss == pytest.approx(ref[0][0], rel=1e-10, abs=1e-15)
    np.testing.assert_allclose(got, d, rtol=1e-9, atol=1e-9 * np.abs(d[:3]).max())


@pytest.mark.parametrize("ns,walls", [(1, False), (2, True)])
def test_states_of_eight_wide_tiles(ns, walls):
    """The recompute's 8 x 8 tiles, which the sizes above do not take."""
    test_reverse_tiles_match_the_complex_step(100, 100, ns, walls)
