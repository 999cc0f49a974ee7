"""The key pass on both sides of the particle density from which its blocks
run in plain order (more than 4096 particles a tile): an ordered set against
the FP64 oracle, and the same set shuffled, which takes other passes or the
other order of atomics, bit for bit (a paint sums whole numbers)."""
import numpy as np
import pytest
import torch

from oracle import pm
from paper_2010_11847_amd import inputs
from paper_2010_11847_amd.binding import PMContext
from tests.gpu_helpers import banner, rel, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_mesh,tiles", [(8, 8), (16, 8), (32, 64)])
@pytest.mark.parametrize("more", [0, 1])
def test_keys_on_both_sides_of_a_dense_tile(gpu, n_mesh, tiles, more):
    n_p = 4096 * tiles + more
    banner(f"keys np={n_p} n={n_mesh}")
    x = inputs.uniform_positions(n_p, n_mesh, seed=n_p)
    c = np.floor(x).astype(np.int64)
    ordered = x[np.argsort((c[:, 0] * n_mesh + c[:, 1]) * n_mesh + c[:, 2], kind="stable")]
    ctx = PMContext(inputs.scaled(inputs.MEDIUM, n_mesh, 8), max_particles=n_p)
    d = ctx.pm_paint(to_dev(ordered))
    assert torch.equal(d, ctx.pm_paint(to_dev(x)))
    assert rel(to_np(d), pm.density_contrast(ordered, n_mesh, n_p)) < 1e-5
