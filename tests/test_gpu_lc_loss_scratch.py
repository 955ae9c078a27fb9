"""The scratch of lc_loss: given by the caller, allocated by the call, or not to be had, in which case the call takes
the form that needs none, as a program that fills the memory expects.

The two forms differ by the rounding of float32 sums of a few hundred terms: 1e-4 of the largest value.
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


@pytest.mark.parametrize("n,count", [(32, 32768), (32, 32769), (64, 2000000)])
def test_scratch(cola, n, count):
    print(f"lc loss scratch n {n} count {count}", file=sys.stderr, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(count)
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda")
    pos = torch.rand((3, count), generator=gen, device="cuda") * 20.0
    df, g1, g3 = rnd(3, n, n, n), rnd(3, count), rnd(3, count)
    stats, d_df = torch.empty(2, dtype=torch.float64, device="cuda"), torch.empty_like(df)
    need = int(cola._lib.lib().cola_lc_loss_workspace_bytes(n, count))
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    want = [t.clone() for t in cola.lc_loss(pos, 20.0, df, g1, g3, stats, d_df, ws)]
    with pytest.raises(cola.ColaError):
        cola.lc_loss(pos, 20.0, df, g1, g3, stats, d_df, ws[:need - 1])
    del ws
    top = float(want[1].abs().max())

    def check():
        d_df.fill_(7.0)
        stats.fill_(7.0)
        cola.lc_loss(pos, 20.0, df, g1, g3, stats, d_df)
        assert torch.allclose(stats, want[0], rtol=1e-12, atol=0.0)
        assert float((d_df - want[1]).abs().max()) <= 1e-4 * top

    check()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (8 << 20)) / total)
    try:
        check()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
