"""How the default launches steps past the caches: the pairs, the marched rows and the single marched steps that it
takes there instead of tiles, on lattices just past each line of the rule and, ragged, on their other side.
Every path does the same arithmetic, so populations have to agree bit for bit with rows marched in a set
shape; wall stresses are FP64 sums in another order (relative 1e-12 of sums of at most 1e5 terms)."""

import numpy as np
import pytest

from cases import make_sim
from test_gpu_tile import case

pytestmark = pytest.mark.gpu

# lx, ly, storage, species, walls, reduce every, two steps per launch, rounding
PATHS = [
    (1793, 760, "f64", 2, False, 0, "auto", None),     # pairs: FP64, two species, periodic, more than 192 MiB
    (1700, 900, "f64", 2, False, 0, "auto", None),     # tiles: narrower
    (1000, 3800, "f64", 2, False, 0, "auto", None),    # pairs: more than 512 MiB
    (3073, 1130, "f64", 2, True, 0, "auto", None),     # marched: FP64, two species, walls
    (1540, 2090, "f64", 2, True, 2, "auto", None),     # marched: reductions
    (2816, 2700, "bf16dev", 2, True, 0, "auto", "stochastic"),  # marched: BF16, more than 256 MiB
    (1500, 3000, "bf16dev", 2, True, 1, "auto", None),          # marched: BF16, reductions
    (1500, 3000, "bf16dev", 1, False, 1, "auto", None),         # tiles: both buffers in the cache
    (1793, 1050, "f32", 2, True, 0, "auto", None),     # tiles, a last single step marched
    (1793, 1050, "f32", 2, True, 1, "auto", None),     # the same with reductions
    (517, 3700, "f32", 2, False, 1, "auto", None),     # tiles: a third of the strips' lanes empty
    (1793, 1050, "f32", 2, False, 0, False, None),     # marched: one step per launch asked for
    (301, 147, "f32", 2, True, 1, False, None),        # tiles of one step: in the cache
]


@pytest.mark.parametrize("lx,ly,storage,ns,walls,every,two,rounding", PATHS)
def test_default_path_is_bitwise_the_marched_rows(lx, ly, storage, ns, walls, every, two, rounding):
    import torch
    c = case(lx, ly, storage, ns, walls)
    print(lx, ly, storage, ns, walls, every, two, rounding, flush=True)
    sims = [make_sim(c, tile=t) for t in (None, (64, 40))]
    for s, sim in enumerate(sims):
        sim.set_two_step(two if s == 0 else False)
        if rounding:
            sim.set_rounding(rounding)
        sim.set_reduce_every(every)
    for n in (1, 2, 3, 5):
        for sim in sims:
            sim.step(n)
        assert torch.equal(sims[0].checkpoint(), sims[1].checkpoint()), n
    if not every:
        sims[0].set_graph(6)
        for sim in sims:
            sim.step(13)
        assert torch.equal(sims[0].checkpoint(), sims[1].checkpoint()), "graph replay"
    if walls and every:
        a, b = (np.array(sim.wall_stress()) for sim in sims)
        assert np.abs(a - b).max() <= 1e-12 * np.abs(b).max()
    for sim in sims:
        sim.close()


@pytest.mark.parametrize("lx,ly,storage,ns,walls", [(2100, 900, "f32", 2, True), (1040, 1030, "f64", 2, False),
                                                    (1500, 1300, "f64", 1, False)])
def test_automatic_pairs_in_a_set_shape(lx, ly, storage, ns, walls):
    """With a launch shape set, the automatic rule pairs the steps of walled FP32 and periodic FP64 lattices beyond
    the Infinity Cache: odd and even counts and graph replay, against the tiles and single marched steps."""
    import torch
    c = case(lx, ly, storage, ns, walls)
    print(lx, ly, storage, ns, walls, flush=True)
    f = []
    for tile, two in ((None, "auto"), ((128, 30), "auto"), ((128, 30), False)):
        sim = make_sim(c, tile=tile)
        sim.set_two_step(two)
        assert sim.two_step_active == (two == "auto")
        sim.step(5)
        sim.set_graph(6)
        sim.step(14)
        f.append(sim.checkpoint())
        sim.close()
    assert torch.equal(f[0], f[1]) and torch.equal(f[0], f[2])
