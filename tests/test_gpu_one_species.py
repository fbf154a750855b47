"""Batches of one species in tiles, which the two-species tests do not instantiate: steps, reductions, graph
replay, totals and fields against marched rows and against contexts of their own, few enough for one tile per
compute unit and more."""

import numpy as np
import pytest

from cases import make_sim
from test_gpu_tile import case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage,walls,rounding", [("f64", False, None), ("f64", True, None), ("f32", False, None),
                                                    ("f32", True, None), ("bf16dev", False, "stochastic"), ("bf16dev", True, None)])
@pytest.mark.parametrize("sizes", [[(61, 37), (20, 9), (40, 33)], [(300, 147), (517, 60), (33, 200), (5, 7)]])
def test_one_species_batches(storage, walls, rounding, sizes):
    import torch
    from paper_1402_6019_amd import Batch
    cases = [dict(case(lx, ly, storage, 1, walls), walls=int(walls), rho_wall=(0.8, 0.0) if walls else (0.0, 0.0),
                  body=(1e-5, 0.0), u_wall=(-0.01, 0.02) if walls else (0.0, 0.0)) for lx, ly in sizes]
    keys = ("g1", "g2", "gab", "body", "rho_wall", "tau", "psi0", "rho0", "rho_ref", "u_wall")
    print(storage, walls, rounding, sizes, flush=True)
    out = []
    for march in (False, True):
        b = Batch([dict({k: c[k] for k in keys}, lx=c["lx"], ly=c["ly"], rho_init=c["rho"]) for c in cases], n_species=1,
                  walls=walls, storage=storage)
        if rounding:
            b.set_rounding(rounding)
        if march:
            b.set_tile(64, 7)
        b.set_graph(10)
        b.step(24)
        b.set_reduce_every(2)
        b.step(5)
        out.append(([b.checkpoint(i) for i in range(b.n)], b.wall_stress() if walls else np.ones(1), b.totals(),
                    [b.moments(i) for i in range(b.n)]))
        b.close()
    assert all(torch.equal(x, y) for x, y in zip(out[0][0], out[1][0]))
    assert np.abs(out[0][1] - out[1][1]).max() <= 1e-12 * np.abs(out[1][1]).max()
    for i, c in enumerate(cases):
        sim = make_sim(c)
        if rounding:
            sim.set_rounding(rounding)
        sim.step(29)
        assert torch.equal(sim.checkpoint(), out[0][0][i])
        assert all(torch.equal(x, y) for x, y in zip(sim.moments(), out[0][3][i]))
        m, p, q = sim.totals()
        assert np.abs(np.array([*m, *p, q]) - out[0][2][i]).max() <= 1e-12 * m[0]  # the same terms, in another order
        sim.close()
