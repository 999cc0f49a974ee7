"""Forces over the mesh sizes at which one workgroup transforms a row of all
three components, from fewer words than threads to the largest, in every cell
residue, against the FP64 oracle."""
import numpy as np
import pytest

from oracle import pm
from paper_2010_11847_amd import inputs
from paper_2010_11847_amd.binding import PMContext
from tests.gpu_helpers import banner, rel, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_mesh", [8, 16, 32, 64, 128, 256])
def test_force_rows_match_oracle(gpu, n_mesh):
    banner(f"force rows n={n_mesh}")
    n_p = 40001
    x = inputs.uniform_positions(n_p, n_mesh, seed=n_mesh)
    c = PMContext(inputs.scaled(inputs.MEDIUM, n_mesh, 8), max_particles=n_p)
    got = to_np(c.pm_force(to_dev(x)))
    want = pm.force(x.astype(np.float64), n_mesh, n_p, 0.3)
    for d in range(3):
        assert rel(got[:, d], want[:, d]) < 1e-5
