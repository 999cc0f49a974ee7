"""Forces and inverse transforms of meshes up to 32^3 keep their bits, which a
run amplifies: the float32 patterns that the library gave when a thread
transformed a whole column (tests/golden/small_mesh_bits.json)."""
import json
import os
from dataclasses import replace

import numpy as np
import pytest
import torch

from paper_2010_11847_amd import inputs
from paper_2010_11847_amd.binding import PMContext
from tests.gpu_helpers import banner

pytestmark = pytest.mark.gpu
with open(os.path.join(os.path.dirname(__file__), "golden", "small_mesh_bits.json")) as fh:
    GOLDEN = json.load(fh)


def bits(a):
    return np.ascontiguousarray(a.cpu().numpy(), np.float32).view(np.uint32).ravel()


@pytest.mark.parametrize("key", sorted(GOLDEN["force"]))
def test_force_bits(gpu, key):
    banner(f"force bits {key}")
    n, deconv, split = (int(v) for v in key.split("/"))
    w = replace(inputs.scaled(inputs.MEDIUM, n, 8), deconv_order=deconv, split_mode=split, split_rs=1.25)
    x = torch.from_numpy(inputs.uniform_positions(24, n, seed=n)).cuda()
    f = PMContext(w, max_particles=512).pm_force(x)
    np.testing.assert_array_equal(bits(f), np.array(GOLDEN["force"][key], np.uint32))


@pytest.mark.parametrize("n", [8, 16, 32, 64])
def test_irfft_bits(gpu, n):
    banner(f"irfft bits n={n}")
    r = np.random.default_rng(n)
    s = (r.standard_normal((n, n, n // 2 + 1)) + 1j * r.standard_normal((n, n, n // 2 + 1))).astype(np.complex64)
    d = PMContext(inputs.scaled(inputs.MEDIUM, n, 8)).pm_irfft(torch.from_numpy(s).cuda())
    i = torch.from_numpy(inputs.sample_indices(n ** 3, 64, seed=n)).cuda()
    np.testing.assert_array_equal(bits(d.view(-1)[i]), np.array(GOLDEN["irfft"][str(n)], np.uint32))
