"""Transforms and mesh force at mesh sides of every kind: powers of two, 3 2^a, 2 3^b and mixtures, so
that every default kernel shape (lines per block that do not divide the side, each radix of the
compile-time plans, each tile width) meets its remainders.  Oracle: numpy's float64 FFTs.

Tolerance: a transform of n^3 values in float32 has a relative RMS error of about eps sqrt(log2 n^3)
(eps = 6e-8): 2e-6 log2(n) holds it with a margin of ten, as in the other transform tests; the force
is two transforms and one product, so twice that.
"""

import math
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1509_04685_amd import workloads as W  # noqa: E402


@pytest.fixture(scope="module")
def cola():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1509_04685_amd as c
    return c


def rms(a):
    return float(np.sqrt(np.mean(np.abs(a) ** 2)))


SIDES = [4, 6, 12, 16, 18, 24, 32, 36, 48, 54, 64, 72, 96, 108, 128, 144, 162, 192, 216, 324]


@pytest.mark.parametrize("n", SIDES)
def test_transforms_and_force(cola, n):
    print(f"mesh side {n}", file=sys.stderr, flush=True)
    x = W.random_field(n, seed=7300 + n, dtype=np.float32)
    xk = np.fft.rfftn(x.astype(np.float64))
    tol = 2e-6 * math.log2(n)
    xd = torch.as_tensor(x, device="cuda")
    got = cola.fft_r2c(xd).cpu().numpy()
    assert rms(got - xk) < tol * rms(xk)
    back = cola.fft_c2r(torch.as_tensor(xk.astype(np.complex64), device="cuda")).cpu().numpy()
    want = x.astype(np.float64) * float(n) ** 3
    assert rms(back - want) < tol * rms(want)
    # the mesh force i k delta_k / k^2 (0 at k = 0 and on each axis's own Nyquist plane)
    box = 100.0
    g = cola.mesh_force(xd, box).cpu().numpy()
    k = 2.0 * np.pi / box * np.fft.fftfreq(n, 1.0 / n)
    kz = 2.0 * np.pi / box * np.fft.rfftfreq(n, 1.0 / n)
    ks = (k[:, None, None], k[None, :, None], kz[None, None, :])
    k2 = ks[0] ** 2 + ks[1] ** 2 + ks[2] ** 2
    k2[0, 0, 0] = np.inf
    for d in range(3):
        kd = np.where(np.abs(ks[d]) > 2.0 * np.pi / box * (n / 2 - 0.5), 0.0, ks[d])
        want = np.fft.irfftn(1j * kd * xk / k2, s=(n, n, n), axes=(0, 1, 2))
        assert rms(g[d] - want) < 2 * tol * rms(want), d
