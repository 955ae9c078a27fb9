"""Cloud-in-cell density where a tile meets very many points: thousands per cell on the smallest meshes, whose tiles
go down to single cells, and clumps of which one tile of a large mesh holds most.

Bound per cell of rho = sum of weights, as in the deposit's other tests: a weight is a product of three factors,
at most 4 roundings of 2^-24, and is rounded to 2^-32; the contrast rho scale - 1 adds one rounding of each:
4e-7 rho scale + 2e-7 + 2.4e-10 scale count.  The sums are integers, so a repeated call gives the same bits.
"""

import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cola():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1509_04685_amd as c
    return c


def density(pos, n, box, least=0.0):
    """(density contrast, sum of weights in its units, number of terms) per cell in float64; weights below `least`
    (a point that rounds up to a node has a fraction of about -1e-7 of its cell coordinate) are raised to it."""
    inv = np.float32(n / box)
    fl = np.floor(pos * inv)
    assert fl.dtype == np.float32
    f = (pos.astype(np.float64) * np.float64(inv) - fl).astype(np.float32).astype(np.float64)
    m = fl.astype(np.int64) % n
    rho, number = np.zeros(n ** 3), np.zeros(n ** 3)
    for c in range(8):
        o = [c >> 2 & 1, c >> 1 & 1, c & 1]
        i = ((m[0] + o[0]) % n * n + (m[1] + o[1]) % n) * n + (m[2] + o[2]) % n
        w = np.ones(pos.shape[1])
        for d in range(3):
            w = w * (f[d] if o[d] else 1.0 - f[d])
        rho += np.bincount(i, weights=np.maximum(w, least), minlength=n ** 3)
        number += np.bincount(i, minlength=n ** 3)
    scale = n ** 3 / pos.shape[1]
    return rho * scale - 1.0, rho * scale, number * scale


@pytest.mark.parametrize("n,count,width", [(2, 100000, 1.0), (3, 300000, 1.0), (5, 400000, 1.0), (6, 120000, 1.0),
                                           (7, 3000000, 1.0), (8, 700000, 1.0), (40, 300000, 0.01), (64, 200000, 0.002),
                                           (130, 1000000, 0.01), (250, 1000000, 0.01), (251, 400000, 0.03)])
def test_density(cola, n, count, width):
    print(f"dense deposit: {count} on {n}^3, width {width}", file=sys.stderr, flush=True)
    box = 50.0
    gen = torch.Generator(device="cuda").manual_seed(n + count)
    if width == 1.0:
        pos = torch.rand((3, count), generator=gen, device="cuda") * box
    else:
        pos = 0.31 * box + width * box * torch.randn((3, count), generator=gen, device="cuda")
        pos[:, ::7] = torch.rand((3, (count + 6) // 7), generator=gen, device="cuda") * box
    pos = torch.remainder(pos, box).contiguous()
    got = cola.cic_density(pos, n, box)
    want, rho, terms = density(pos.cpu().numpy(), n, box)
    err = np.abs(got.cpu().numpy().astype(np.float64).reshape(-1) - want)
    worst = float((err / (4e-7 * rho + 2e-7 + 2.4e-10 * terms)).max())
    assert worst <= 1.0, worst
    assert torch.equal(cola.cic_density(pos, n, box), got)


# one block sorts up to 4096 points on up to 8192 keys (8 per tile: 6912 on 96^3, 9464 on 104^3), the general path more
@pytest.mark.parametrize("n,count", [(2, 1), (2, 4096), (3, 4097), (16, 4096), (16, 4097), (96, 4096), (96, 4097),
                                     (104, 4096), (33, 1), (64, 1023), (64, 1025)])
def test_few_points(cola, n, count):
    print(f"few points: {count} on {n}^3", file=sys.stderr, flush=True)
    box = 50.0
    gen = torch.Generator(device="cuda").manual_seed(n + count)
    pos = torch.rand((3, count), generator=gen, device="cuda") * box
    got = cola.cic_density(pos, n, box)
    want, rho, terms = density(pos.cpu().numpy(), n, box)
    err = np.abs(got.cpu().numpy().astype(np.float64).reshape(-1) - want)
    assert np.all(err <= 4e-7 * rho + 2e-7 + 2.4e-10 * terms)
    if n in (16, 64, 96):  # pm_fields keeps the sign of a weight
        want, rho, terms = density(pos.cpu().numpy(), n, box, least=-1.0)
        rho = np.abs(rho)
        fields = cola.pm_fields(pos, n, box, g=False, acc=False)["delta"].cpu().numpy().astype(np.float64).reshape(-1)
        assert np.all(np.abs(fields - want) <= 4e-7 * rho + 2e-7 + 2.4e-10 * terms)
