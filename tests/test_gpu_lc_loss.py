"""The tiled adjoint of the correction's loss against the form with atomics to memory, which the float64
oracle checks elsewhere: sides that no tile divides, few and many particles per cell, residuals that are
zero, infinite or NaN, and a zero denominator.

Bound: both forms add c float32 terms w r s per cell and component.  The atomic form rounds each running
sum (2^-24 of it), the tiled one each term to 2^-30 of the largest (at most 2^20 particles here) and
the result once, so they differ by at most (c + 4) 2^-24 of the sum of |terms| and c 2^-30 of the largest.
"""

import ctypes
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


def make(n, count, seed, box=20.0):
    rng = np.random.default_rng(seed)
    pos = rng.uniform(0.0, box, size=(3, count))
    k = count // 2
    pos[:, :k] = box / 2 + rng.normal(0.0, 0.05 * box, size=(3, k))
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a, dtype=np.float32), device="cuda")
    g1 = rng.normal(size=(3, count))
    return (t(np.mod(pos, box)), box, t(rng.normal(size=(3, n, n, n)) * 0.3), t(g1),
            t(g1 + rng.normal(size=(3, count)) * 0.5))


def atomic(cola, pos, box, df, g1, g3):
    n = df.shape[-1]
    stats = torch.empty(2, dtype=torch.float64, device="cuda")
    out = torch.empty_like(df)
    p3 = lambda a: (ctypes.c_void_p * 3)(*[a[d].data_ptr() for d in range(3)])
    s = cola._lib.lib().cola_lc_loss(n, box, p3(pos), pos.shape[1], p3(df), p3(g1), p3(g3),
                                     ctypes.c_void_p(stats.data_ptr()), ctypes.c_void_p(out.data_ptr()),
                                     ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert s == 0
    return stats, out


def spread(pos, box, n, values):
    """Sum over particles of w * value per cell, float64."""
    u = pos.cpu().numpy().astype(np.float64) * (n / box)
    m = np.floor(u).astype(np.int64)
    f = u - m
    out = np.zeros(n ** 3)
    for c in range(8):
        o = [c >> 2 & 1, c >> 1 & 1, c & 1]
        i = ((m[0] + o[0]) % n * n + (m[1] + o[1]) % n) * n + (m[2] + o[2]) % n
        w = np.prod([np.abs(f[d] if o[d] else 1 - f[d]) for d in range(3)], axis=0)
        out += np.bincount(i, weights=w * values, minlength=n ** 3)
    return out


@pytest.mark.parametrize("n,count", [(2, 3), (5, 200), (8, 4000), (10, 1), (16, 5003), (21, 30000), (33, 2000),
                                     (48, 200000)])
def test_tiled_loss(cola, n, count):
    print(f"lc loss n {n} count {count}", file=sys.stderr, flush=True)
    args = make(n, count, 100 * n + count)
    ws, wd = atomic(cola, *args)
    stats, d_df = cola.lc_loss(*args)
    assert torch.allclose(stats, ws, rtol=1e-12, atol=0.0)
    terms = 2.0 / float(ws[1]) * 12.0  # no |r| above 12 by far: g, dF and target are of order 1
    number = spread(args[0], args[1], n, np.ones(count))
    c = np.ceil(8 * number) + 8
    bound = (c + 4) * 2.0 ** -24 * number * terms + c * 2.0 ** -30 * terms
    err = (d_df - wd).abs().amax(dim=0).cpu().numpy().reshape(-1)
    assert np.all(err <= bound + 1e-30), float((err / (bound + 1e-30)).max())


def test_tiled_loss_special_values(cola):
    n, count = 16, 3000
    for case in ("inf", "nan", "same"):
        print(f"lc loss special {case}", file=sys.stderr, flush=True)
        pos, box, df, g1, g3 = make(n, count, 7)
        if case == "inf":
            g3[1, 17] = float("inf")
        elif case == "nan":
            g1[2, 1234] = float("nan")
        else:
            g3 = g1.clone()  # zero denominator
        ws, wd = atomic(cola, pos, box, df, g1, g3)
        stats, d_df = cola.lc_loss(pos, box, df, g1, g3)
        assert torch.equal(torch.isfinite(stats), torch.isfinite(ws))
        assert torch.equal(torch.isnan(d_df), torch.isnan(wd))
        fin = torch.isfinite(wd)
        assert torch.equal(torch.isfinite(d_df), fin)
        assert torch.allclose(d_df[fin], wd[fin], rtol=1e-4, atol=1e-6)
    # residuals of exactly zero: g1 = g3 - G[dF] with dF = 0
    pos, box, df, g1, g3 = make(n, count, 8)
    g3[:, 100:] = g1[:, 100:]
    g3[:, :100] = g1[:, :100] + 1.0
    df.zero_()
    ws, wd = atomic(cola, pos, box, df, g1, g3)
    stats, d_df = cola.lc_loss(pos, box, df, g1, g3)
    assert torch.allclose(d_df, wd, rtol=1e-5, atol=1e-9)
