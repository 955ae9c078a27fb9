"""Cloud-in-cell density on mesh sides that no tile side divides, against a float64 sum.

The mesh is cut into tiles whose last one along a side may be narrower; a cell on the upper face of
a tile (the last layer of the mesh included) also belongs to the next tile up, across the periodic
edge.  Sides around multiples of the tile sides, sides smaller than one tile, odd sides past 256,
and counts from a few points to hundreds per cell (which take the small tiles) cover the edges.

The reference takes the cell of the float32 product x (n / L) and the fraction of its exact value,
rounded once, with a weight of -1e-7 (a product that rounds up to a node) cut to 0.  Bound per cell of the density rho = sum of weights: a weight is a product of
three factors, at most 4 roundings of 2^-24, plus 2^-32 of fixed point; the contrast
rho scale - 1 adds one rounding of each.  So |error| <= 4e-7 rho scale + 2e-7 + 2.4e-10 scale count.
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


@pytest.mark.parametrize("n,count", [(2, 5), (3, 100), (5, 40), (7, 2000), (8, 1), (9, 700), (15, 3000), (17, 50000),
                                     (23, 10), (24, 400000), (31, 60000), (33, 700), (34, 300000), (63, 5000),
                                     (65, 200000), (72, 30000), (100, 20000), (127, 1000000), (250, 30000),
                                     (257, 3000)])
def test_density_of_ragged_sides(cola, n, count):
    print(f"density {count} points on {n}^3", file=sys.stderr, flush=True)
    rng = np.random.default_rng(1000 * n + count)
    box = 37.5
    pos = rng.uniform(0.0, box, size=(3, count))
    pos[:, : count // 3] = box / 2 + rng.normal(0.0, 0.02 * box, size=(3, count // 3))
    pos = np.mod(pos, box).astype(np.float32)
    pos[pos >= np.float32(box)] = 0.0
    pos[:, 0] = 0.0                                    # on a node
    pos[:, -1] = np.nextafter(np.float32(box), np.float32(0))  # in the last cell, next to the periodic edge
    got = cola.cic_density(torch.as_tensor(pos, device="cuda"), n, box).cpu().numpy().astype(np.float64)
    h = np.float32(n / box)
    fl = np.floor(pos * h)
    assert fl.dtype == np.float32
    f = (pos.astype(np.float64) * np.float64(h) - fl).astype(np.float32).astype(np.float64)
    m = fl.astype(np.int64) % n
    rho = np.zeros(n ** 3)
    number = np.zeros(n ** 3)
    for a in (0, 1):
        for b in (0, 1):
            for c in (0, 1):
                i = (((m[0] + a) % n) * n + (m[1] + b) % n) * n + (m[2] + c) % n
                w = (f[0] if a else 1 - f[0]) * (f[1] if b else 1 - f[1]) * (f[2] if c else 1 - f[2])
                rho += np.bincount(i, weights=np.maximum(w, 0.0), minlength=n ** 3)
                number += np.bincount(i, minlength=n ** 3)
    scale = n ** 3 / count
    err = np.abs(got.reshape(-1) - (rho * scale - 1.0))
    assert np.all(err <= 4e-7 * rho * scale + 2e-7 + 2.4e-10 * scale * number), float(err.max())
    # bitwise repeatable
    again = cola.cic_density(torch.as_tensor(pos, device="cuda"), n, box).cpu().numpy()
    assert np.array_equal(again.astype(np.float64), got)


@pytest.mark.parametrize("n,count,same", [(16, 3000, True), (36, 46656, True), (16, 60000, False)])
def test_fields_density(cola, n, count, same):
    """The density of pm_fields: the tiled deposit while its records fit the workspace (about a particle
    per cell), the same to the bit; float atomics beyond, where a sum of c weights below 1 in any order is
    off by at most c 2^-24 of its value, c < 200 here."""
    print(f"pm_fields density {count} points on {n}^3", file=sys.stderr, flush=True)
    rng = np.random.default_rng(n + count)
    pos = torch.as_tensor(rng.uniform(0.0, 10.0, size=(3, count)).astype(np.float32), device="cuda").clamp_(max=9.9999)
    want = cola.cic_density(pos, n, 10.0)
    got = cola.pm_fields(pos, n, 10.0, g=False, acc=False)["delta"]
    if same:
        assert torch.equal(got, want)
    else:
        assert float((got - want).abs().max()) < 200 * 6e-8 * float(want.max() + 1.0)
