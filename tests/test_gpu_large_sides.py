"""Transforms and mesh force on the large mesh sides whose default kernels no tuning and no workload picks, up to
1296^3: every one has its own radix sequence, values per thread and exchange pads.

The field is a sum of three products u(x) v(y) w(z) of random sequences: every value and every mode differs from
zero, and its spectrum is the sum of the products of 1D transforms, which numpy gives in float64.

Tolerance: as for the smaller sides, 2e-6 log2(n) relative RMS for a transform, twice that for the force (two
transforms and a product), which is compared by its transform, one more.
"""

import math
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

SLAB = 16


@pytest.fixture(scope="module")
def cola():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1509_04685_amd as c
    return c


def product(a, b, c, x0, x1):
    """sum_r a_r[x] b_r[y] c_r[z] for x0 <= x < x1."""
    return sum(a[r, x0:x1, None, None] * (b[r, :, None] * c[r, None, :]) for r in range(a.shape[0]))


def filled(parts, n, m, dtype):
    out = torch.empty((n, n, m), dtype=dtype, device="cuda")
    for x in range(0, n, SLAB):
        out[x:x + SLAB] = product(*parts, x, min(n, x + SLAB)).to(dtype)
    return out


def off(got, want, n):
    """Relative RMS of got - want(x0, x1)."""
    err = torch.zeros((), dtype=torch.float64, device="cuda")
    size = torch.zeros_like(err)
    for x in range(0, n, SLAB):
        w = want(x, min(n, x + SLAB))
        err += torch.sum(torch.abs(got[x:x + SLAB].to(w.dtype) - w) ** 2)
        size += torch.sum(torch.abs(w) ** 2)
    return math.sqrt(float(err) / float(size))


@pytest.mark.parametrize("n", [432, 486, 576, 648, 864, 972, 1024, 1152, 1296])
def test_large_side(cola, n):
    print(f"large mesh side {n}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(9100 + n)
    real = rng.normal(size=(3, 3, n))
    dev = lambda a: torch.as_tensor(a, device="cuda")
    x_parts = [dev(p) for p in real]
    k_parts = [dev(np.fft.fft(real[0])), dev(np.fft.fft(real[1])), dev(np.fft.rfft(real[2]))]
    tol = 2e-6 * math.log2(n)
    xd = filled(x_parts, n, n, torch.float32)
    assert off(cola.fft_r2c(xd), lambda a, b: product(*k_parts, a, b), n) < tol
    spec = filled(k_parts, n, n // 2 + 1, torch.complex64)
    assert off(cola.fft_c2r(spec), lambda a, b: product(*x_parts, a, b) * float(n) ** 3, n) < tol
    del spec
    # the mesh force i k delta_k / k^2 (0 at k = 0 and on each axis's own Nyquist plane)
    box = 100.0
    k = 2.0 * np.pi / box * np.fft.fftfreq(n, 1.0 / n)
    kz = 2.0 * np.pi / box * np.fft.rfftfreq(n, 1.0 / n)
    axes = [dev(k)[:, None, None], dev(k)[None, :, None], dev(kz)[None, None, :]]
    nyquist = 2.0 * np.pi / box * (n / 2 - 0.5)
    g = cola.mesh_force(xd, box)
    del xd
    for d in range(3):
        kd = torch.where(axes[d].abs() > nyquist, 0.0, axes[d])

        def force(a, b):
            kx = axes[0][a:b]
            k2 = kx ** 2 + axes[1] ** 2 + axes[2] ** 2
            if a == 0:
                k2[0, 0, 0] = 1.0  # k_d is 0 there
            return 1j * ((kd[a:b] if d == 0 else kd) / k2) * product(*k_parts, a, b)

        assert off(cola.fft_r2c(g[d]), force, n) < 3 * tol, d
    del g
    torch.cuda.empty_cache()
