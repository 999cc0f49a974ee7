"""The forward transform of measured spectra, bit for bit.  A mesh that is
zero off the line y = z = 0 passes the z and y transforms without a rounding,
so every (ky, kz) of its spectrum holds the x transform of that line, and a
host transform with the same roundings (fmaf where the kernel fuses) has to
give the same bits; P(k) is then the float64 sum over those values."""
import ctypes
import ctypes.util

import numpy as np
import pytest
import torch

from paper_2010_11847_amd import inputs
from paper_2010_11847_amd.binding import PMContext
from tests.gpu_helpers import banner

pytestmark = pytest.mark.gpu

F = np.float32
fmaf = ctypes.CDLL(ctypes.util.find_library("m")).fmaf
fmaf.restype = ctypes.c_float
fmaf.argtypes = [ctypes.c_float] * 3
# below 64 points the levels are those of a whole column, whichever threads share them
STAGES = {8: (8, 1), 16: (16, 1), 32: (32, 1), 64: (8, 8), 128: (16, 8), 256: (16, 16), 512: (32, 16), 1024: (32, 32)}


def twiddle(x, y, idx, eighth_as_others):
    """(x + i y) exp(-2 pi i idx / 32), idx < 16."""
    if idx == 0:
        return x, y
    if idx == 8:
        return y, F(-x)
    c, s = F(np.cos(2 * np.pi * idx / 32)), F(-np.sin(2 * np.pi * idx / 32))
    if idx > 8 or (idx == 4 and eighth_as_others):
        re = fmaf(-y, s, F(x * c))
    else:
        re = fmaf(x, c, F(-F(y * s)))
    im = fmaf(x, s, F(y * c)) if idx == 4 and not eighth_as_others else fmaf(y, c, F(x * s))
    return F(re), F(im)


def stage(v, second):
    r = len(v)
    size = r
    while size > 1:
        half = size // 2
        for s in range(0, r, size):
            for k in range(half):
                (ax, ay), (bx, by) = v[s + k], v[s + k + half]
                v[s + k] = F(ax + bx), F(ay + by)
                v[s + k + half] = twiddle(F(ax - bx), F(ay - by), k * (32 // size),
                                          second and (r == 8 or s + size < r))
        size = half
    bits = r.bit_length() - 1
    return [v[int(format(i, f"0{bits}b")[::-1], 2) if bits else 0] for i in range(r)]


def column(line, stages):
    n, (r1, r2) = len(line), stages
    tw = [(F(np.cos(2 * np.pi * k / n)), F(-np.sin(2 * np.pi * k / n))) for k in range(n)]
    mid = [[None] * r2 for _ in range(r1)]
    for j in range(r2):
        v = stage([(F(line[r2 * i + j]), F(0)) for i in range(r1)], False)
        for l, (x, y) in enumerate(v):
            if l and r2 > 1:
                wx, wy = tw[j * l]
                x, y = F(fmaf(x, wx, F(-F(y * wy)))), F(fmaf(x, wy, F(y * wx)))
            mid[l][j] = x, y
    out = np.empty(n, np.complex64)
    for l in range(r1):
        for l2, (x, y) in enumerate(stage(mid[l], True)):
            out[l + r1 * l2] = x + 1j * y
    return out


def line_mesh(n):
    line = np.random.default_rng(n).standard_normal(n).astype(F)
    d = torch.zeros((n, n, n), device="cuda")
    d[:, 0, 0] = torch.from_numpy(line).cuda()
    return line, d


@pytest.mark.parametrize("n", [8, 16, 32, 64, 128, 256, 512, 1024])
def test_rfft_bits(gpu, n):
    banner(f"rfft bits n={n}")
    line, d = line_mesh(n)
    f = torch.from_numpy(column(line, STAGES[n])).cuda()
    s = PMContext(inputs.scaled(inputs.MEDIUM, n, 8)).pm_rfft(d)
    assert bool((torch.view_as_real(s) == torch.view_as_real(f)[:, None, None, :]).all())


@pytest.mark.parametrize("n,deconv", [(8, False), (16, True), (32, False), (64, True), (128, False), (256, False),
                                      (512, True)])
def test_power_digits(gpu, n, deconv):
    """Float64 sums of at most 2e6 positive terms, in any order, agree to 1e-12."""
    banner(f"power digits n={n} deconv={deconv}")
    w = inputs.scaled(inputs.MEDIUM, n, 8)
    line, d = line_mesh(n)
    x = column(line, STAGES[n]).astype(np.complex128)
    f = np.fft.fftfreq(n, 1 / n)
    fy, fz = f[:, None], np.arange(n // 2 + 1)[None, :]
    win = np.sinc(f / n) ** 2
    wz = np.sinc(np.arange(n // 2 + 1) / n) ** 2
    if deconv:   # the window tables are float32
        win, wz = win.astype(F).astype(np.float64), wz.astype(F).astype(np.float64)
    weight = np.where((fz == 0) | (fz == n // 2), 1.0, 2.0) + 0 * fy
    p, m = np.zeros(n // 2 + 1), np.zeros(n // 2 + 1)
    for i in range(n):
        b = np.floor(np.sqrt(f[i] ** 2 + fy ** 2 + fz ** 2) + 0.5).astype(int)
        t = weight * abs(x[i]) ** 2 / ((win[i] * win[:, None] * wz[None, :]) ** 2 if deconv else 1.0)
        ok = b <= n // 2
        p += np.bincount(b[ok], t[ok], n // 2 + 1)
        m += np.bincount(b[ok], weight[ok], n // 2 + 1)
    _, pk, modes = PMContext(w).pm_power(d, deconv=deconv)
    np.testing.assert_array_equal(modes, m[1:])
    np.testing.assert_allclose(pk, p[1:] / m[1:] * w.box_size ** 3 / n ** 6, rtol=1e-12)
