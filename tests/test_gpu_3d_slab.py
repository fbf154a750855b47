"""Slabs of few planes: the split step where a population buffer fits the Infinity Cache, the march past it,
without a field of psi then; both bitwise the kernel of a set launch shape."""

import numpy as np
import pytest

import lbgen

pytestmark = pytest.mark.gpu


def make(lx, ly, lz, storage, ns, walls, tile=None):
    from paper_1402_6019_amd import Sim3
    a = np.random.default_rng(lx + ly).uniform(0.3, 1.1, (lz, ly, lx))
    rho = np.stack([a, 1.4 - a])[:ns]
    kw = dict(body=(1e-5, 0.0, 2e-5), rho_wall=lbgen.EMULSION_POOR) if walls else {}
    return Sim3(lx, ly, lz, rho, n_species=ns, walls=walls, storage=storage, g1=lbgen.EMULSION_G1, g2=lbgen.EMULSION_G2,
                gab=lbgen.EMULSION_GAB, rho0=lbgen.EMULSION_RHO0, tau=(0.9, 1.2), rho_ref=(0.7, 0.7), tile=tile, **kw)


SLABS = [(lx, ly, lz, *mode) for lx, ly, lz in [(300, 203, 7), (517, 515, 8), (1030, 517, 5)]
         for mode in [("f32", 2, False), ("f64", 1, True), ("f64", 2, True)]]
SLABS += [(5, 600000, 5, "f32", 1, False), (5, 400000, 5, "f32", 2, True)]  # more rows than a grid has


@pytest.mark.parametrize("lx,ly,lz,storage,ns,walls", SLABS)
def test_slab_is_bitwise_the_set_shape(lx, ly, lz, storage, ns, walls):
    import torch
    print(lx, ly, lz, storage, ns, walls, flush=True)
    sims = [make(lx, ly, lz, storage, ns, walls, tile=t) for t in (None, (4, 8))]
    for sim in sims:
        sim.step(3)
    assert torch.equal(sims[0].checkpoint(), sims[1].checkpoint())
    for x, y in zip(sims[0].moments(), sims[1].moments()):
        assert torch.equal(x, y)
    for sim in sims:
        sim.close()


def test_z_planes_of_nearly_4_gib():
    """A plane that ends less than 1 MiB below 4 GiB: the lanes past a ragged strip's end neither read nor write."""
    import torch
    lx, ly, lz = 5, 882900, 5  # rows of 19 x 64 values
    assert 2**32 - 2**20 < 19 * 64 * 4 * ly < 2**32
    f = []
    for tile in (None, (4, 8)):
        sim = make(lx, ly, lz, "f32", 1, False, tile=tile)
        print(tile, flush=True)
        sim.step(2)
        f.append(sim.checkpoint())
        sim.close()
        del sim
    assert torch.equal(*f)


def test_slab_past_the_cache_holds_no_field():
    import torch
    lx, ly, lz = 1024, 1024, 5  # 760 MiB per buffer; a field would take 84 MB
    make(64, 48, 8, "f32", 2, False).close()  # loads the kernels

    def held():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[1] - torch.cuda.mem_get_info()[0] - torch.cuda.memory_reserved()

    before = held()
    sim = make(lx, ly, lz, "f32", 2, False)
    assert held() - before < 16 * lx * ly * lz / 2
    sim.close()
