"""Painting and forces of particles in any order: sets around the size from
which an unknown order is looked at, in an ordered, a scattered and a lopsided
form (each sorted by another path), against the FP64 oracle."""
import numpy as np
import pytest

from oracle import pm
from paper_2010_11847_amd import inputs
from paper_2010_11847_amd.binding import PMContext
from tests.gpu_helpers import banner, rel, to_dev, to_np

pytestmark = pytest.mark.gpu
FIRST = 1 << 17   # particles from which the order is looked at


def positions(kind, n_p, n_mesh):
    if kind == "scattered":
        return inputs.uniform_positions(n_p, n_mesh, seed=n_p)
    if kind == "lopsided":   # most of the particles in one clump: a bucket of many times the mean
        return inputs.clustered_positions(n_p, n_mesh, seed=n_p, n_clumps=1, width=0.8, frac=0.9)
    x = inputs.uniform_positions(n_p, n_mesh, seed=n_p)   # ordered: by cell, z fastest
    c = np.floor(x).astype(np.int64)
    return x[np.argsort((c[:, 0] * n_mesh + c[:, 1]) * n_mesh + c[:, 2], kind="stable")]


@pytest.mark.parametrize("kind", ["scattered", "lopsided", "ordered"])
@pytest.mark.parametrize("n_p,n_mesh", [(FIRST - 1, 64), (FIRST, 64), (FIRST + 4097, 32), (3 * FIRST + 1, 128)])
def test_force_in_any_order_matches_oracle(gpu, n_p, n_mesh, kind):
    banner(f"force np={n_p} n={n_mesh} {kind}")
    x = positions(kind, n_p, n_mesh)
    c = PMContext(inputs.scaled(inputs.MEDIUM, n_mesh, 8), max_particles=n_p)
    d = to_np(c.pm_paint(to_dev(x)))
    assert rel(d, pm.density_contrast(x, n_mesh, n_p)) < 1e-5
    assert rel(to_np(c.pm_force(to_dev(x))), pm.force(x.astype(np.float64), n_mesh, n_p, 0.3)) < 1e-5


@pytest.mark.parametrize("kind", ["scattered", "lopsided"])
def test_many_particles_in_any_order(gpu, kind):
    n_p, n_mesh = (1 << 23) + 3, 128
    banner(f"paint np={n_p} {kind}")
    x = positions(kind, n_p, n_mesh)
    c = PMContext(inputs.scaled(inputs.MEDIUM, n_mesh, 8), max_particles=n_p)
    assert rel(to_np(c.pm_paint(to_dev(x))), pm.density_contrast(x, n_mesh, n_p)) < 1e-5
    f = to_np(c.pm_force(to_dev(x)))
    idx = inputs.sample_indices(n_p, 2000, seed=1)
    green = [pm.force_mesh(pm.rfftn(pm.density_contrast(x, n_mesh, n_p)), pm.green_function(n_mesh, 0.3), d, n_mesh)
             for d in range(3)]
    assert rel(f[idx], np.stack([pm.readout(m, x[idx]) for m in green], 1)) < 1e-5
