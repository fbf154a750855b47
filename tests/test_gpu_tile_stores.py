"""The store policies in 32 x 16 tiles, two workgroups per compute unit, the only shape with a streaming
variant: every storage mode and rounding, one, two and three steps per launch, with and without reductions,
ragged on both sides, against each other and against marched rows; and batches beyond the Infinity Cache,
which stream by themselves.  Populations bit for bit; wall stresses at one shape too, as the policy does not
change the order of their sums."""

import numpy as np
import pytest

from cases import make_sim
from test_gpu_tile import case

pytestmark = pytest.mark.gpu

MODES = [("f64", 1, False, None), ("f64", 2, True, None), ("f32", 1, True, None), ("f32", 2, False, None),
         ("f32", 2, True, None), ("bf16dev", 2, True, None), ("bf16dev", 1, False, "stochastic"),
         ("bf16dev", 2, False, "stochastic"), ("bf16dev", 2, True, "stochastic")]


@pytest.mark.parametrize("storage,ns,walls,rounding", MODES)
@pytest.mark.parametrize("every,two", [(0, "auto"), (1, "auto"), (3, "auto"), (1, False)])
def test_streaming_tiles(storage, ns, walls, rounding, every, two):
    import torch
    c = case(517, 270, storage, ns, walls)
    if ns == 1 and walls:
        c.update(walls=1, rho_wall=(0.8, 0.0), body=(1e-5, 0.0), u_wall=(-0.01, 0.02))
    print(storage, ns, walls, rounding, every, two, flush=True)
    f, w = [], []
    for tile, policy in ((None, "write_through"), (None, "streaming"), (None, "auto"), ((64, 7), "auto")):
        sim = make_sim(c, tile=tile)
        sim.set_store_policy(policy)
        sim.set_two_step(two)
        sim.set_reduce_every(every)
        if rounding:
            sim.set_rounding(rounding)
        for n in (1, 2, 5):
            sim.step(n)
        f.append(sim.checkpoint())
        w.append(sim.wall_stress() if walls and every else None)
        sim.close()
    assert all(torch.equal(f[0], x) for x in f[1:])
    assert w[0] == w[1] == w[2]


@pytest.mark.parametrize("storage,ns,walls", [("f64", 2, True), ("f64", 1, False), ("f32", 2, True)])
def test_streaming_batches(storage, ns, walls):
    """Buffers of 165 MiB and more: FP64 streams in every launch, FP32 in launches of one step."""
    import torch
    from paper_1402_6019_amd import Batch
    each = {("f64", 2): 5, ("f64", 1): 10, ("f32", 2): 10}[storage, ns]
    cases = [case(1000 - 7 * i, 260 + i, storage, ns, walls) for i in range(each)]
    keys = ("g1", "g2", "gab", "body", "rho_wall", "tau", "psi0", "rho0", "rho_ref", "u_wall")
    print(storage, ns, walls, flush=True)
    out = []
    for march in (False, True):
        b = Batch([dict({k: c[k] for k in keys if k in c}, lx=c["lx"], ly=c["ly"], rho_init=c["rho"]) for c in cases],
                  n_species=ns, walls=walls, storage=storage)
        assert b.pop_bytes > 128 << 20
        if march:
            b.set_tile(64, 40)
        for n, every in ((1, 0), (4, 0), (1, 1), (3, 1)):
            b.set_reduce_every(every)
            b.step(n)
        out.append(([b.checkpoint(i) for i in range(b.n)], b.wall_stress() if walls else np.ones(1)))
        b.close()
    assert all(torch.equal(x, y) for x, y in zip(out[0][0], out[1][0]))
    assert np.abs(out[0][1] - out[1][1]).max() <= 1e-12 * np.abs(out[1][1]).max()
