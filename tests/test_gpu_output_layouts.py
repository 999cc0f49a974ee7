"""Real outputs off the 16-byte grid, which leave through the library's own
layout and must hold the same bits as aligned ones, and the transforms of the
largest meshes against float64."""
import ctypes as C
from dataclasses import replace

import numpy as np
import pytest
import torch

from paper_2010_11847_amd import inputs
from paper_2010_11847_amd.binding import PMContext
from tests.gpu_helpers import banner

pytestmark = pytest.mark.gpu


def ptr(t):
    return C.c_void_p(t.data_ptr())


def off_grid(shape):
    t = torch.full((int(np.prod(shape)) + 2,), float("nan"), device="cuda")
    v = t[1:-1].view(shape)
    assert v.data_ptr() % 16 == 4
    return t, v


@pytest.mark.parametrize("n", [8, 32, 128])
def test_irfft_into_an_unaligned_mesh(gpu, n):
    banner(f"irfft unaligned n={n}")
    c = PMContext(inputs.scaled(inputs.MEDIUM, n, 8))
    g = torch.Generator(device="cuda").manual_seed(n)
    s = torch.fft.rfftn(torch.randn((n, n, n), generator=g, device="cuda")).contiguous()
    buf, out = off_grid((n, n, n))
    assert c.lib.pm_irfft(c.ctx, ptr(s), ptr(out)) == 0
    assert torch.equal(out, c.pm_irfft(s))
    assert buf[0].isnan() and buf[-1].isnan()


@pytest.mark.parametrize("n,order", [(8, 2), (64, 1), (64, 2)])
def test_noise_cotangent_into_an_unaligned_array(gpu, n, order):
    banner(f"adjoint unaligned n={n} order={order}")
    w = replace(inputs.scaled(inputs.ADJ_SMALL, n, n, n_steps=2), lpt_order=order)
    c = PMContext(w)
    noise = c.pm_noise(5)
    pos, mom = c.pm_init_lpt(0, w.a_list[0], noise=noise)
    ck = torch.empty((len(w.a_list), 2, w.n_particles, 3), device="cuda")
    c.pm_run(w.a_list, pos, mom, ckpt=ck)
    gd = torch.rand((n,) * 3, device="cuda", generator=torch.Generator("cuda").manual_seed(1)) - 0.5
    want = c.pm_run_adjoint(w.a_list, ck, noise=noise, grad_delta=gd)
    a = np.ascontiguousarray(w.a_list, dtype=np.float64)
    gx, gp = torch.zeros_like(pos), torch.zeros_like(mom)
    buf, gn = off_grid((n, n, n))
    assert c.lib.pm_run_adjoint(c.ctx, a.ctypes.data_as(C.POINTER(C.c_double)), len(a), ptr(ck), ptr(noise), ptr(gd),
                                ptr(gx), ptr(gp), ptr(gn)) == 0
    for x, y in zip(want, (gx, gp, gn)):
        assert torch.equal(x, y)
    assert buf[0].isnan() and buf[-1].isnan()


def norm(x):
    """Norm in float64, plane by plane (a float64 copy of the whole would not fit beside it)."""
    return sum(float((torch.view_as_real(p) if p.is_complex() else p).double().square().sum()) for p in x) ** 0.5


@pytest.mark.parametrize("n", [512, 1024])
def test_large_transforms(gpu, n):
    """Float32 transforms of 3 log2 n radix-2 levels: at most about
    3 log2(n) 2^-24 = 2e-6 of the norm (in practice a tenth)."""
    banner(f"transforms n={n}")
    c = PMContext(inputs.scaled(inputs.MEDIUM, n, 8))
    x = torch.randn((n, n, n), generator=torch.Generator(device="cuda").manual_seed(n), device="cuda")
    s = c.pm_rfft(x)
    # whole (ky, kz) planes of the float64 transform at some kx
    for kx in (0, 1, n // 2, n - 3):
        phase = torch.exp(-2j * np.pi * kx / n * torch.arange(n, device="cuda", dtype=torch.float64))
        plane = torch.zeros((n, n), dtype=torch.complex128, device="cuda")
        for i in range(n):
            plane += phase[i] * x[i].double()
        ref = torch.fft.fft2(plane)[:, : n // 2 + 1]
        assert float((s[kx] - ref).abs().square().sum().sqrt() / ref.abs().square().sum().sqrt()) < 2e-6
    assert norm(c.pm_irfft(s) - x) / norm(x) < 4e-6
