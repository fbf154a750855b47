"""The tile step (several time steps per launch, states in between on chip) against the row-marching
step, at the edges of its dispatch: every tile shape, ragged last tiles, lattices narrower than a
tile's neighbourhood, remainders of the steps per launch, every storage mode.  The per-site
arithmetic is the same expressions in the same order, so populations have to agree bit for bit; wall
stresses are FP64 sums in another order (relative 1e-12 of sums of at most 1e5 terms)."""

import numpy as np
import pytest

import lbgen
from cases import film_case, make_sim

pytestmark = pytest.mark.gpu

# lx, ly: 4x8 tiles (one and several wraps of a narrow lattice), 16x8, 16x16 and 32x16 tiles
SIZES = [(5, 5), (9, 41), (160, 5), (64, 64), (61, 37), (131, 130), (301, 147), (517, 270)]


def case(lx, ly, storage, ns, walls):
    if ns == 1:
        return film_case(lx, ly, seed=lx, storage=storage, tau=0.9)
    # the emulsion couplings on random densities between the two phases (any lattice size)
    a = np.random.default_rng(lx + ly).uniform(0.3, 1.1, (ly, lx))
    c = dict(film_case(lx, ly, storage=storage, tau=1.1), ns=2, walls=int(walls), g1=lbgen.EMULSION_G1, g2=lbgen.EMULSION_G2,
             gab=lbgen.EMULSION_GAB, body=(1e-5, 0.0), rho_wall=lbgen.EMULSION_POOR if walls else (0.0, 0.0),
             rho0=lbgen.EMULSION_RHO0, rho=np.stack([a, 1.4 - a]), rho_ref=(0.7, 0.7))
    if walls:
        c["u_wall"] = (-0.01, 0.02)
    return c


def populations(c, steps, tile=None, rounding=None, cross=False, graph=0):
    sim = make_sim(dict(c, cross_psi=cross), tile=tile)
    if rounding:
        sim.set_rounding(rounding)
    if graph:
        sim.set_graph(graph)
    out = []
    for n in steps:
        sim.step(n)
        out.append(sim.checkpoint().cpu().numpy())
    sim.close()
    return out


@pytest.mark.parametrize("lx,ly", SIZES)
@pytest.mark.parametrize("storage,ns,walls", [("f64", 1, False), ("f64", 2, True), ("f32", 2, False), ("f32", 2, True),
                                              ("bf16dev", 2, True)])
def test_tile_steps_are_bitwise_the_marched_steps(lx, ly, storage, ns, walls):
    c = case(lx, ly, storage, ns, walls)
    steps = (1, 2, 3, 4, 5)
    print(lx, ly, storage, ns, walls, flush=True)
    for a, b in zip(populations(c, steps), populations(c, steps, tile=(64, 7))):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("lx,ly", [(100, 100), (127, 129)])
@pytest.mark.parametrize("storage,ns,walls", [("f64", 1, False), ("f64", 2, True), ("f32", 2, True), ("bf16dev", 2, False)])
def test_eight_wide_tiles(lx, ly, storage, ns, walls):
    """8 x 8 tiles, ragged: lattices whose 4 x 8 tiles are more than the compute units."""
    c = case(lx, ly, storage, ns, walls)
    print(lx, ly, storage, ns, walls, flush=True)
    for a, b in zip(populations(c, (1, 2, 3, 4, 5)), populations(c, (1, 2, 3, 4, 5), tile=(64, 7))):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("lx,ly", [(400, 300), (320, 200)])
@pytest.mark.parametrize("storage,ns,walls", [("f64", 1, False), ("f64", 2, True), ("f32", 2, True), ("bf16dev", 2, False)])
def test_wide_tiles_of_one_per_compute_unit(lx, ly, storage, ns, walls):
    """32 x 16 tiles that fit the compute units one each: three steps per launch (FP64 with two
    species: two), ragged on both sides and on one."""
    c = case(lx, ly, storage, ns, walls)
    print(lx, ly, storage, ns, walls, flush=True)
    for a, b in zip(populations(c, (1, 2, 3, 4, 5)), populations(c, (1, 2, 3, 4, 5), tile=(64, 7))):
        assert np.array_equal(a, b)


def test_tile_steps_with_other_options():
    c = case(61, 37, "bf16dev", 2, True)
    a, b = (populations(c, (7,), tile=t, rounding="stochastic") for t in (None, (64, 7)))
    assert np.array_equal(a[0], b[0])
    a, b = (populations(c, (10, 10, 3), tile=t, rounding="stochastic", graph=10) for t in (None, (64, 7)))
    assert all(np.array_equal(x, y) for x, y in zip(a, b)), "graph replay, stochastic rounding"
    for ns, walls in ((1, False), (2, True)):
        c = case(131, 40, "f32", ns, walls)
        a, b = (populations(c, (8, 5, 8), tile=t, cross=ns == 2, graph=4) for t in (None, (64, 7)))
        assert all(np.array_equal(x, y) for x, y in zip(a, b)), "graph replay, cross term over psi"


@pytest.mark.parametrize("lx,ly", [(61, 37), (301, 147)])
@pytest.mark.parametrize("every", [1, 2, 5])
def test_tile_steps_reduce_as_marched_steps(lx, ly, every):
    c = case(lx, ly, "f32", 2, True)
    got = []
    for tile in (None, (64, 7)):
        sim = make_sim(c, tile=tile)
        sim.set_reduce_every(every)
        for n in (1, 4, 6):
            sim.step(n)
        got.append((np.array(sim.wall_stress()), sim.checkpoint().cpu().numpy()))
        sim.close()
    assert np.array_equal(got[0][1], got[1][1])
    scale = np.abs(got[1][0]).max()
    assert np.abs(got[0][0] - got[1][0]).max() <= 1e-12 * scale


def test_autotune_takes_the_faster_of_tile_and_march():
    """Either way the populations stay bitwise those of the other."""
    c = case(131, 130, "f32", 2, True)
    sim = make_sim(c)
    sim.autotune(trial_steps=3)
    sim.step(5)
    f = sim.checkpoint().cpu().numpy()
    sim.close()
    assert np.array_equal(f, populations(c, (5,), tile=(64, 7))[0])


@pytest.mark.parametrize("storage,rounding", [("f64", None), ("f32", None), ("bf16dev", "stochastic")])
@pytest.mark.parametrize("sizes", [[(61, 37), (20, 9), (40, 33)], [(300, 147), (517, 60), (33, 200), (5, 7)]])
def test_batch_tile_steps_are_bitwise_the_marched_steps(storage, rounding, sizes):
    """Instances of uneven sizes, few enough for one tile per compute unit and more; reductions and
    graph replay too."""
    from paper_1402_6019_amd import Batch
    cases = [case(lx, ly, storage, 2, True) for lx, ly in sizes]
    keys = ("g1", "g2", "gab", "body", "rho_wall", "tau", "psi0", "rho0", "rho_ref", "u_wall")
    out = []
    for march in (False, True):
        b = Batch([dict({k: c[k] for k in keys}, lx=c["lx"], ly=c["ly"], rho_init=c["rho"]) for c in cases], n_species=2,
                  walls=True, storage=storage)
        if rounding:
            b.set_rounding(rounding)
        if march:
            b.set_tile(64, 7)
        b.set_graph(10)
        b.step(24)
        b.set_reduce_every(2)
        b.step(5)
        out.append(([b.checkpoint(i).cpu().numpy() for i in range(b.n)], b.wall_stress()))
        b.close()
    assert all(np.array_equal(x, y) for x, y in zip(out[0][0], out[1][0]))
    assert np.abs(out[0][1] - out[1][1]).max() <= 1e-12 * np.abs(out[1][1]).max()
