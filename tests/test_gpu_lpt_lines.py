"""LPT initial conditions over the line lengths of the z stages (less than one
workgroup's words, one round of them, several; with and without the second
order), off the lattice's cell corners, with the displacement fields of the
COLA frame, against the FP64 oracle."""
from dataclasses import replace

import numpy as np
import pytest

from oracle import lpt, pm
from oracle.rng import white_noise
from paper_2010_11847_amd import inputs
from paper_2010_11847_amd.binding import PMContext
from tests.gpu_helpers import banner, rel, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_part,ratio,order", [(8, 1, 2), (8, 2, 1), (16, 1, 2), (64, 1, 2), (128, 1, 2), (128, 1, 1),
                                                (256, 1, 2)])
def test_particles_and_frame_match_oracle(gpu, n_part, ratio, order):
    banner(f"lpt np={n_part} ratio={ratio} order={order}")
    n_mesh = n_part * ratio
    w = replace(inputs.scaled(inputs.MEDIUM, n_mesh, n_part), lpt_order=order, lattice_shift=0.25)
    c = PMContext(w)
    psi1, psi2 = c.pm_set_lpt_frame()
    pos, mom = c.pm_init_lpt(w.seed, w.a_list[0])
    dk = lpt.linear_field_k(white_noise(w.seed, n_part), w.box_size, w.cosmo, False)
    s1, s2 = lpt.lpt_displacements(dk, 2)
    x, p = lpt.initial_state(s1, s2, w.a_list[0], n_mesh, w.cosmo.omega_m, order, 0.25)
    gx = to_np(pos)
    assert gx.min() >= 0 and gx.max() < n_mesh
    assert np.abs(pm.min_image(gx - x, n_mesh)).max() < 1e-4 * max(1.0, n_mesh / 64)
    assert rel(to_np(mom), p) < 1e-5
    assert rel(to_np(psi1), ratio * s1.reshape(-1, 3)) < 1e-5
    if order >= 2:
        assert rel(to_np(psi2), ratio * s2.reshape(-1, 3)) < 1e-5
    else:
        assert not psi2.any()
