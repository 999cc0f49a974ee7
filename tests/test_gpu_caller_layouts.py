"""Transforms that read and write the caller's meshes and spectra directly:
a buffer off the 16-byte grid takes a copy through the library's own layout
instead and must give the same bits; the binned spectrum at every bin count
and mode cut against the FP64 oracle."""
import numpy as np
import pytest
import torch

from oracle import power
from paper_2010_11847_amd import inputs
from paper_2010_11847_amd.binding import PMContext
from tests.gpu_helpers import banner, rel, to_np

pytestmark = pytest.mark.gpu


def off_grid(t):
    """The same values in a contiguous tensor 4 bytes off the 16-byte grid."""
    buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    buf[1:] = t.reshape(-1)
    return buf[1:].view(t.shape)


@pytest.mark.parametrize("n", [8, 64, 128])
def test_unaligned_meshes_give_the_same_bits(gpu, n):
    banner(f"unaligned meshes n={n}")
    c = PMContext(inputs.scaled(inputs.MEDIUM, n, n))
    g = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn((n, n, n), generator=g, device="cuda")
    y = off_grid(x)
    assert y.data_ptr() % 16 == 4
    assert torch.equal(torch.view_as_real(c.pm_rfft(x)), torch.view_as_real(c.pm_rfft(y)))
    assert torch.equal(torch.cat(c.pm_init_lpt(0, 0.1, noise=x)), torch.cat(c.pm_init_lpt(0, 0.1, noise=y)))
    out = torch.empty_like(x)
    assert torch.equal(torch.cat(c.pm_init_lpt(0, 0.1, noise=x)), torch.cat(c.pm_init_lpt(0, 0.1, noise=y, noise_out=out)))
    assert torch.equal(out, x)
    for a, b in zip(c.pm_power(x), c.pm_power(y)):
        np.testing.assert_allclose(a, b, rtol=1e-12)


@pytest.mark.parametrize("n,n_bins,n_max,deconv", [(8, 4, 0, True), (16, 3, 0, False), (32, 16, 9, True),
                                                  (128, 64, 0, True), (128, 1, 0, False), (256, 100, 64, False)])
def test_binned_power_matches_oracle(gpu, n, n_bins, n_max, deconv):
    banner(f"power n={n} bins={n_bins} nmax={n_max} deconv={deconv}")
    w = inputs.scaled(inputs.MEDIUM, n, 8)
    d = inputs.normal_array((n, n, n), seed=n)
    k, p, m = PMContext(w).pm_power(torch.from_numpy(d).cuda(), n_bins=n_bins, n_max=n_max, deconv=deconv)
    ok, op, om = power.power(d.astype(np.float64), w.box_size, n_bins=n_bins, deconvolve_cic=deconv, n_max=n_max)
    np.testing.assert_array_equal(m, om)
    full = om > 0
    assert rel(k[full], ok[full]) < 1e-12 and rel(p[full], op[full]) < 1e-5
    assert to_np(torch.from_numpy(p[~full])).sum() == 0
