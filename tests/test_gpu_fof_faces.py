"""Friends across the faces of the cells of the friends-of-friends grid, against the oracle (bit-exact).

A particle looks into a neighbouring cell only where a friend can reach that far, so partners are placed on
both sides of cell faces, edges and corners and of the box's own faces, at distances just below and above the
linking length, in every direction; grids of one cell, of three, four and of several linking lengths per
cell, and one pile of thousands of particles in one cell that spans many blocks of records.
"""

import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import fof as F  # noqa: E402


@pytest.fixture(scope="module")
def cola():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1509_04685_amd as c
    return c


# (particles, box, linking length): the grid has min(floor(box / (1.001 link)), ceil(cbrt(n))) cells per side
@pytest.mark.parametrize("n,box,link", [(40, 10.0, 4.0), (3000, 10.0, 3.3), (3000, 10.0, 2.4), (6000, 40.0, 0.35),
                                        (30000, 100.0, 0.62), (30000, 1000.0, 30.0)])
def test_faces(cola, n, box, link):
    print(f"fof faces n {n} box {box} link {link}", file=sys.stderr, flush=True)
    rng = np.random.default_rng(n + int(link * 100))
    nc = int(min(np.floor(box / (link * 1.001)), np.ceil(np.cbrt(n))))
    cell = box / max(nc, 1)
    m = n // 2
    base = rng.uniform(0.0, box, size=(3, m))
    on = rng.random((3, m)) < 0.6  # put these coordinates within 1e-4 of a face (the box's own among them)
    face = rng.integers(0, max(nc, 1) + 1, size=(3, m)) * cell
    base = np.where(on, face + rng.normal(0.0, 1e-4 * cell, size=(3, m)), base)
    v = rng.normal(size=(3, m))
    v /= np.linalg.norm(v, axis=0)
    mate = base + v * link * rng.choice([0.2, 0.97, 0.9999, 1.0001, 1.03], size=m)
    pos = np.mod(np.concatenate([base, mate, rng.uniform(0.0, box, size=(3, n - 2 * m))], axis=1), box)
    pos = np.ascontiguousarray(pos[:, rng.permutation(n)], dtype=np.float32)
    pos[pos >= np.float32(box)] = 0.0
    g, s = cola.fof(torch.as_tensor(pos, device="cuda"), box, link)
    og, os_ = F.fof(pos, box, link)
    assert np.array_equal(g.cpu().numpy(), og)
    assert np.array_equal(s.cpu().numpy(), os_)


def test_pile(cola):
    print("fof pile", file=sys.stderr, flush=True)
    rng = np.random.default_rng(3)
    n, box, link = 9000, 30.0, 0.3
    pos = rng.uniform(0.0, box, size=(3, n))
    k = 5000  # a chain of clumps around one cell, some of them joined
    pos[:, :k] = 15.0 + rng.normal(0.0, 0.5, size=(3, k))
    pos = np.ascontiguousarray(pos[:, rng.permutation(n)], dtype=np.float32)
    g, s = cola.fof(torch.as_tensor(pos, device="cuda"), box, link)
    og, os_ = F.fof(pos, box, link)
    assert np.array_equal(g.cpu().numpy(), og)
    assert np.array_equal(s.cpu().numpy(), os_)
    cat = cola.fof_catalogue(torch.as_tensor(pos, device="cuda"), box, g, s, 2, 1.0,
                             cola.fof_workspace(n, box, link))
    want = F.catalogue(pos, box, og, os_, 2, 1.0)
    assert np.array_equal(cat["root"].cpu().numpy(), want["root"])
    assert np.array_equal(cat["n"].cpu().numpy(), want["n"])
    # float64 sums of up to n offsets below box / 2 in any order
    assert np.abs(cat["com"].cpu().numpy() - want["com"]).max() < n * box * 2.0 ** -52
