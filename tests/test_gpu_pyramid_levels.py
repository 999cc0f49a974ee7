"""REDUCE and EXPAND at the edges of their tiles (the smallest coarse grids,
up to four levels) through the pyramid force and its transpose, and force
checkpoints that lie off the 16-byte grid."""
import numpy as np
import pytest
import torch

from oracle import adjoint as A
from oracle import pyramid as P
from oracle.rng import white_noise
from paper_2010_11847_amd import inputs
from paper_2010_11847_amd.binding import PMContext
from tests.gpu_helpers import banner, rel, to_dev, to_np
from tests.test_gpu_adjoint import SIGMA, gpu_grad_along, oracle_trajectory
from tests.test_gpu_pyramid import OM, wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_mesh,levels", [(16, 1), (32, 2), (64, 3), (128, 4), (64, 1)])
def test_pyramid_force_at_every_depth(gpu, n_mesh, levels):
    banner(f"pyramid force n={n_mesh} levels={levels}")
    n_p = 20001
    x = inputs.clustered_positions(n_p, n_mesh, seed=n_mesh + levels)
    g = to_np(PMContext(wl(n_mesh, 8, levels), max_particles=n_p).pm_force(to_dev(x)))
    assert rel(g, P.force(x.astype(np.float64), n_mesh, n_p, OM, levels=levels)) < 1e-5


@pytest.mark.parametrize("n_mesh,levels", [(16, 1), (64, 3)])
def test_pyramid_adjoint_at_the_smallest_coarse_grid(gpu, n_mesh, levels):
    banner(f"pyramid adjoint n={n_mesh} levels={levels}")
    w = wl(n_mesh, n_mesh // 2, levels, a_list=inputs.a_linear(0.1, 1.0, 2))
    noise = white_noise(w.seed, w.n_part)
    xs = oracle_trajectory(w, noise, force_fn=lambda x: P.force(x, n_mesh, w.n_particles, OM, levels=levels))
    target = inputs.normal_array((n_mesh,) * 3, seed=3).astype(np.float64)
    g = gpu_grad_along(w, xs, noise, target)
    assert rel(g, A.grad_along_trajectory(xs, noise, w, target, SIGMA, pyramid_levels=levels)) < 1e-4


def test_unaligned_force_checkpoints_give_the_same_run(gpu):
    banner("pyramid run with force checkpoints off the 16-byte grid")
    w = wl(32, 16, 1, a_list=inputs.a_linear(0.1, 1.0, 3))
    out = []
    for shift in (0, 1):
        c = PMContext(w)
        buf = torch.empty(4 * 32 ** 3 * 3 + shift, device="cuda")
        c.pm_set_force_ckpt(4, buf[shift:])
        pos, mom = c.pm_init_lpt(w.seed, w.a_list[0])
        c.pm_run(w.a_list, pos, mom)
        out.append((pos, mom, buf[shift:]))
    for a, b in zip(*out):
        assert torch.equal(a, b)
