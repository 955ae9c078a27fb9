"""The density of pm_fields, cell by cell, where cells outnumber the particles by far and where particles
sit on the mesh's nodes, whose fractions round to either side of zero.

The weights are formed in float64 from the fractions as the deposit defines them: the cell from the float32
product u = x n / L, the fraction x n / L - floor(u) of the exact product, rounded once; it is negative
where u rounds up to a node.  Bound per cell of c terms: each weight is a product of three factors (1 - f rounded
once) in float32, 5 2^-24 of it, each addition rounds once, and so does the contrast:
(c + 5) 2^-24 cells / particles * sum |w| + 2^-24 max(|delta|, 1).
"""

import sys

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cola():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1509_04685_amd as c
    return c


def cells_and_fractions(pos, n, box):
    inv = torch.tensor(n / box, dtype=torch.float64).to(torch.float32).to("cuda")
    fl = torch.floor(pos * inv)
    f = (pos.double() * inv.double() - fl.double()).float()
    return torch.remainder(fl.long(), n), f


def density(pos, n, box):
    """(density contrast, sum of |weights|, number of terms) per cell in float64."""
    m, f = cells_and_fractions(pos, n, box)
    out = [torch.zeros(n ** 3, dtype=torch.float64, device="cuda") for _ in range(3)]
    for c in range(8):
        o = [c >> 2 & 1, c >> 1 & 1, c & 1]
        i = ((m[0] + o[0]) % n * n + (m[1] + o[1]) % n) * n + (m[2] + o[2]) % n
        w = torch.ones_like(f[0], dtype=torch.float64)
        for d in range(3):
            w = w * (f[d].double() if o[d] else 1.0 - f[d].double())
        for a, v in zip(out, (w, w.abs(), torch.ones_like(w))):
            a.index_add_(0, i, v)
    scale = n ** 3 / pos.shape[1]
    return out[0] * scale - 1.0, out[1] * scale, out[2]


@pytest.mark.parametrize("n,count,where", [(384, 40000, "anywhere"), (128, 300, "anywhere"), (48, 50000, "anywhere"),
                                           (96, 100000, "nodes"), (54, 40000, "nodes")])
def test_fields_density(cola, n, count, where):
    print(f"fields deposit: {count} on {n}^3, {where}", file=sys.stderr, flush=True)
    box = 100.1
    gen = torch.Generator(device="cuda").manual_seed(n + count)
    if where == "nodes":
        pos = (torch.randint(0, n, (3, count), generator=gen, device="cuda").double() * (box / n)).float()
    else:
        pos = torch.rand((3, count), generator=gen, device="cuda") * box
    got = cola.pm_fields(pos, n, box, g=False, acc=False)["delta"].double().reshape(-1)
    want, size, terms = density(pos, n, box)
    bound = 2.0 ** -24 * ((terms + 5.0) * size + want.abs().clamp(min=1.0))
    worst = float(((got - want).abs() / bound).max())
    assert worst <= 1.0, worst


@pytest.mark.parametrize("n,count", [(32, 40000), (48, 40000), (48, 100)])
def test_positions_that_are_not_finite(cola, n, count):
    """A NaN or infinite coordinate, or one beyond float32 once in cells, makes the eight cells that it reaches
    and the force NaN or infinite, on either side of the size at which the deposit changes its form; NaN falls into
    cell 0, infinity into that of the largest int32."""
    box = 1.0
    big = (2 ** 31 - 1) % n
    small = (-(2 ** 31)) % n
    for value, cell in ((float("nan"), 0), (float("inf"), big), (float("-inf"), small), (3e38, big)):
        print(f"fields deposit: {value} among {count} on {n}^3", file=sys.stderr, flush=True)
        gen = torch.Generator(device="cuda").manual_seed(count)
        pos = torch.rand((3, count), generator=gen, device="cuda") * box
        pos[:, 57] = torch.tensor([4.25, 5.5, (n - 1) + 0.75], device="cuda") / n
        pos[1, 57] = value
        out = cola.pm_fields(pos, n, box, acc=False)
        want = torch.zeros((n, n, n), dtype=torch.bool, device="cuda")
        for x in (4, 5):
            for y in (cell, (cell + 1) % n):
                for z in (n - 1, 0):
                    want[x, y, z] = True
        assert torch.equal(~torch.isfinite(out["delta"]), want)
        assert not bool(torch.isfinite(out["g"]).any())
    out = cola.pm_fields(torch.rand((3, count), device="cuda") * box, n, box, acc=False)
    assert bool(torch.isfinite(out["delta"]).all()) and bool(torch.isfinite(out["g"]).all())
