"""The adjoint's checkpoints on lattices whose rows are padded: no more workspace than FP64 copies of the sites'
populations and what the sweep needs beside them take, and the same gradient whether a segment is recomputed or
was kept (the recomputed states are bitwise the states stepped through, and every sum adds the same terms in
the same order)."""

import pytest

from cases import make_sim
from test_gpu_tile import case

pytestmark = pytest.mark.gpu


def bound(lx, ly, ns, T, every, reverse):
    """Bytes of every segment's start as FP64 sites, a buffer (rows of 256, FP64), two segments of fields and
    rows at the walls, lambda twice, and 1 MiB of the rest."""
    n = lx * ly
    segments = -(-T // every)
    return (segments * 72 * ns * n + 72 * ns * -(-lx // 256) * 256 * ly + 2 * every * (8 * reverse * n + 144 * ns * lx) +
            2 * 9 * ns * n * reverse + (1 << 20))


@pytest.mark.parametrize("lx,ly,storage,ns,walls,fp64", [(5, 900, "f64", 2, True, False), (64, 40, "f64", 1, False, False),
                                                        (61, 37, "f32", 2, True, True), (300, 70, "f32", 2, True, False),
                                                        (61, 37, "bf16dev", 1, False, False), (256, 33, "f64", 2, True, False)])
def test_recomputed_segments(lx, ly, storage, ns, walls, fp64):
    from paper_1402_6019_amd import _binding as B
    c = case(lx, ly, storage, ns, walls)
    c["body"] = (3e-5, 0.0)
    T, lw = 37, (1.0 if walls else 0.0, 0.3)
    print(lx, ly, storage, ns, walls, fp64, flush=True)
    got = []
    for every in (4, 1, 5):
        sim = make_sim(c)
        if every > 1:
            need = sim._lib.lb_adjoint_workspace_bytes(sim._h, T, every, B.LB_ADJ_FP64 if fp64 else 0)
            assert need <= bound(lx, ly, ns, T, every, 8 if fp64 or storage == "f64" else 4)
        loss, g = sim.adjoint(T, lw, every=every, fp64_reverse=fp64)
        got.append((loss, *g))
        f = sim.checkpoint()
        if every == 4:
            first = f
        assert bool((f == first).all())
        sim.close()
    assert got[0] == got[1] == got[2]
