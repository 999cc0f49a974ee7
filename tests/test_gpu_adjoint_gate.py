"""The reverse sweep's last point: with a momentum cotangent of zero its
launches return at once, with any other value they run.  A cotangent too small
to move any result (1e-30 of one particle against cotangents of order one)
takes the other way through the sweep and gives the same numbers."""
from dataclasses import replace

import pytest
import torch

from paper_2010_11847_amd import inputs
from paper_2010_11847_amd.binding import PMContext
from tests.gpu_helpers import banner

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_mesh,n_part,fck,deconv", [(16, 16, False, 0), (64, 32, True, 0), (64, 32, False, 2),
                                                      (128, 64, False, 0)])
def test_zero_and_tiny_momentum_cotangents_agree(gpu, n_mesh, n_part, fck, deconv):
    banner(f"adjoint gate n={n_mesh} np={n_part} fck={fck} deconv={deconv}")
    w = replace(inputs.scaled(inputs.ADJ_SMALL, n_mesh, n_part, n_steps=3), deconv_order=deconv)
    c = PMContext(w)
    if fck:
        c.pm_set_force_ckpt(len(w.a_list))
    noise = c.pm_noise(5)
    pos, mom = c.pm_init_lpt(0, w.a_list[0], noise=noise)
    ck = torch.empty((len(w.a_list), 2, w.n_particles, 3), device="cuda")
    c.pm_run(w.a_list, pos, mom, ckpt=ck)
    gd = torch.rand((n_mesh,) * 3, device="cuda", generator=torch.Generator("cuda").manual_seed(1)) - 0.5
    tiny = torch.zeros((w.n_particles, 3), device="cuda")
    tiny[-1, 1] = 1e-30
    a = c.pm_run_adjoint(w.a_list, ck, noise=noise, grad_delta=gd)
    b = c.pm_run_adjoint(w.a_list, ck, noise=noise, grad_delta=gd, grad_mom=tiny)
    for x, y in zip(a, b):
        assert torch.isfinite(x).all() and x.abs().max() > 0
        assert torch.equal(x, y)
    # the counts that the gated paints left: a paint equals a new context's
    assert torch.equal(c.pm_paint(pos), PMContext(w).pm_paint(pos))
