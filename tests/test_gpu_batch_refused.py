"""A launch shape that lb_batch_set_tile refuses leaves the batch as it was: its steps, its graphs and the
buffer they alternate between."""

import numpy as np
import pytest

import lbgen

pytestmark = pytest.mark.gpu


def test_refused_shape_changes_nothing():
    """Nine instances whose strips of one row are more than the 2^20 workgroups a shape may have.  A replay of
    ten steps is five launches of two, so it also swaps the buffers."""
    import torch
    from paper_1402_6019_amd import Batch
    rho = lbgen.uniform_noise(65, 65535, 1.0, 0.01, seed=7)[None]
    small = lbgen.uniform_noise(33, 20, 1.0, 0.01, seed=8)[None]
    kw = dict(g1=(lbgen.FILM_G1, 0.0), g2=(lbgen.FILM_G2, 0.0), tau=(0.9, 0.9), psi0=1.0, rho0=1.0, rho_ref=(1.0, 0.0))
    inst = [dict(kw, lx=33, ly=20, rho_init=small)] + [dict(kw, lx=65, ly=65535, rho_init=rho)] * 9
    out = []
    for disturb in (False, True):
        b = Batch(inst, n_species=1, walls=False, storage="bf16dev")
        b.set_graph(10)
        b.step(10)
        shape = b.get_tile()
        if disturb:
            with pytest.raises(Exception, match="too many tiles"):
                b.set_tile(64, 1, 3)
        b.step(10)
        out.append([b.checkpoint(i) for i in (0, 1)])
        kept = b.get_tile() == shape
        b.close()
    assert torch.equal(out[0][0], out[1][0])
    assert torch.equal(out[0][1], out[1][1])
    assert kept
