"""P(k) and multipoles where rows end inside a run of modes, where the shells outnumber the LDS bins, and where
the last shell cuts runs off.

Rows of 4, 6, 18 and 36 modes end in a run of fewer than eight, 72 in a whole one; 1100 shells are summed in
global memory, n / 2 and 3 in LDS.  Mode counts are equal and mean |k| agrees to 1e-12.  Power: the
oracle starts from the same positions in float32, whose rounding turns a mode by up to pi 72 2^-24 = 1.4e-5, as
much as the float32 deposit and transform add: with e = 1.5e-5 a mode is off by 2 sqrt(P P_max) e <=
1e-3 P + 2.3e-7 P_max, taken as 1e-3 P + 1e-5 P_max (times 9, the largest 2 l + 1, for the multipoles).
"""

import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import cola as ocola, cosmology as ocosmo, power as opower  # noqa: E402


@pytest.fixture(scope="module")
def cola():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1509_04685_amd as c
    return c


@pytest.mark.parametrize("n_pk,n_bins", [(4, 2), (6, 1100), (18, 9), (18, 3), (36, 1100), (36, 18), (72, 36), (72, 3)])
def test_runs(cola, n_pk, n_bins):
    print(f"P(k) runs n_pk {n_pk} n_bins {n_bins}", file=sys.stderr, flush=True)
    from paper_1509_04685_amd import workloads as W
    box = 100.0
    prob = cola.make_problem(box, 12, 1, 19.0, 3)
    cosmo = cola.make_cosmology(**W.COSMOLOGY)
    a = float(ocola.Schedule(ocola.Problem(box, 12, 1, 19.0, 3), ocosmo.Cosmology(**W.COSMOLOGY)).a[1])
    st = cola.ParticleState(prob)
    ws = cola.Workspace(prob, n_pk=n_pk)
    cola.ic_2lpt(prob, cosmo, [11], st, ws)
    cola.step(prob, cosmo, st, 1, ws)
    pos = cola.positions(prob, st).cpu().numpy().astype(np.float64)
    for los in (0, 1, 2):
        got = [t.cpu().numpy()[0] for t in cola.power_multipoles(prob, cosmo, st, a, n_pk, n_bins, ws, los=los,
                                                                 redshift_space=False)]
        ref = opower.multipoles(pos, n_pk, box, n_bins, los)
        assert np.array_equal(got[4], ref[4])
        some = ref[4] > 0
        assert np.allclose(got[0][some], ref[0][some], rtol=1e-12, atol=0)
        p0 = np.abs(ref[1][some])
        bound = 1e-3 * p0 + 1e-5 * p0.max()
        assert np.all(np.abs(got[1][some] - ref[1][some]) <= bound)
        for ell in (2, 3):
            assert np.all(np.abs(got[ell][some] - ref[ell][some]) <= 9 * bound), (los, ell)
    km, pk, nm = [t.cpu().numpy()[0] for t in cola.power_spectrum(prob, cosmo, st, a, n_pk, n_bins, ws)]
    assert np.array_equal(nm, ref[4])
    assert np.allclose(km[some], ref[0][some], rtol=1e-12, atol=0)
    assert np.allclose(pk[some], got[1][some], rtol=1e-10, atol=0)
