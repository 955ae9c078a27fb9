"""The scan of the counts per key, at the edges of its three forms: one block (up to 16384 keys), blocks that add
up the sums before them (up to 4096 blocks of 4096 keys), sums scanned in a pass of their own.

Deposits reach the first two: a CIC density is right only if every record sits in its own slot.  Points on
lattice sites give whole cells, so the density is exact.  The third takes a friends-of-friends grid
past 16.8e6 cells: pairs of points on a lattice, far from all others, whose groups are known.
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


# keys: 8 per tile of 8 x 8 x 16 cells at two points per cell: 64, 1000, 8192 and 16384 (one block); 20808, 34848
@pytest.mark.parametrize("n", [16, 40, 96, 128, 136, 168])
def test_density_of_sites(cola, n):
    print(f"key scan: sites of {n}^3", file=sys.stderr, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n)
    cell = torch.randint(0, n ** 3, (2 * n ** 3,), generator=gen, device="cuda")
    pos = torch.stack([cell // (n * n), (cell // n) % n, cell % n]).to(torch.float32)
    got = cola.cic_density(pos, n, float(n))
    want = torch.bincount(cell, minlength=n ** 3).to(torch.float64) * 0.5 - 1.0
    assert torch.equal(got.reshape(-1).to(torch.float64), want)


def test_pairs_on_a_large_grid(cola):
    print("key scan: pairs on 210^3 sites", file=sys.stderr, flush=True)
    s = 210
    n = 2 * s ** 3  # 265^3 cells
    gen = torch.Generator(device="cuda").manual_seed(5)
    slot = torch.randperm(n, generator=gen, device="cuda")  # place of point i: site slot // 2, mate slot % 2
    site = slot // 2
    pos = torch.stack([site // (s * s), (site // s) % s, site % s]).to(torch.float32)
    pos[2] += 0.3 * (slot % 2).to(torch.float32)
    group, size = cola.fof(pos, float(s), 0.5)
    at = torch.empty_like(slot)
    at[slot] = torch.arange(n, device="cuda")
    first = torch.minimum(at[slot], at[slot ^ 1])
    assert torch.equal(group.to(torch.int64), first)
    assert bool((size[first] == 2).all())
