"""The tiled adjoint of the correction's loss where residuals differ by orders of magnitude: between regions,
inside one cell, between components, and one particle against all others.

The box has one unit per cell, so cells and fractions are exact, and the residuals are given (zero correction and
target), so the terms w r of a cell are known in float64.  Bound: that of float32 sums, which it has to keep at
any spread: for c terms (c + 8) 2^-24 of their sum of magnitudes (weights and terms rounded as products,
additions, the factor 2 / D, the result).  Cells that no residual reaches are exactly zero.
"""

import ctypes
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


def loss_with_workspace(cola, pos, box, df, g1, g3):
    lib, n, count = cola._lib.lib(), df.shape[-1], pos.shape[1]
    stats = torch.empty(2, dtype=torch.float64, device="cuda")
    out = torch.empty_like(df)
    p3 = lambda a: (ctypes.c_void_p * 3)(*[a[d].data_ptr() for d in range(3)])
    need = lib.cola_lc_loss_workspace_bytes(n, count)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    assert lib.cola_lc_loss_ws(n, box, p3(pos), count, p3(df), p3(g1), p3(g3), ctypes.c_void_p(stats.data_ptr()),
                               ctypes.c_void_p(out.data_ptr()), ctypes.c_void_p(ws.data_ptr()), need,
                               ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    return stats, out


def residuals(kind, pos, n, gen):
    r = torch.randn(pos.shape, generator=gen, device="cuda")
    if kind == "regions":
        r[:, pos[0] < 0.5 * n] *= 1e-6
    elif kind == "mixed":
        r *= 10.0 ** -(8.0 * torch.rand(pos.shape[1], generator=gen, device="cuda"))
    elif kind == "components":
        r *= torch.tensor([[1.0], [1e-7], [1e-12]], device="cuda")
    elif kind == "outlier":
        r[:, 1:] *= 1e-9
        r[:, 0] = torch.tensor([1e6, -3.0, 0.0], device="cuda")
    elif kind == "extremes":
        r *= torch.where(pos[1] < 0.5 * n, 1e18, 1e-18)
    return r


@pytest.mark.parametrize("kind", ["regions", "mixed", "components", "outlier", "extremes"])
@pytest.mark.parametrize("n,count", [(2, 3), (3, 70000), (16, 5003), (21, 60000), (48, 200000)])
def test_spread_of_residuals(cola, n, count, kind):
    print(f"lc loss range {kind} n {n} count {count}", file=sys.stderr, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n + count)
    pos = torch.rand((3, count), generator=gen, device="cuda") * n
    pos[:, :count // 4] = 0.5 * n + 0.1 * (pos[:, :count // 4] - 0.5 * n)
    r = residuals(kind, pos, n, gen)
    zero = torch.zeros((3, n, n, n), device="cuda")
    args = (pos, float(n), zero, r, torch.zeros_like(r))
    m = torch.floor(pos)
    f = pos - m
    sums = torch.zeros((3, n ** 3), dtype=torch.float64, device="cuda")
    size = torch.zeros_like(sums)
    terms = torch.zeros(n ** 3, dtype=torch.float64, device="cuda")
    for c in range(8):
        o = [c >> 2 & 1, c >> 1 & 1, c & 1]
        i = (m.long() + torch.tensor(o, device="cuda")[:, None]) % n
        i = (i[0] * n + i[1]) * n + i[2]
        w = torch.ones(count, dtype=torch.float64, device="cuda")
        for d in range(3):
            w = w * (f[d].double() if o[d] else 1.0 - f[d].double())
        sums.index_add_(1, i, w * r.double())
        size.index_add_(1, i, (w * r.double()).abs())
        terms.index_add_(0, i, torch.ones_like(w))
    D = float((r.double() ** 2).sum())
    for name, got in (("workspace", loss_with_workspace(cola, *args)), ("lc_loss", cola.lc_loss(*args))):
        stats, d_df = got
        assert abs(float(stats[1]) / D - 1.0) < 1e-12
        assert abs(float(stats[0]) - 1.0) < 1e-12
        err = (d_df.double().reshape(3, -1) - sums * (2.0 / D)).abs()
        bound = (terms + 8.0) * 2.0 ** -24 * size * (2.0 / D) + 1e-45
        worst = float((err / bound).max())
        assert worst <= 1.0, (name, worst)
