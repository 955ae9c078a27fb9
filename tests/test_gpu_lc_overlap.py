"""Backward passes of one network that overlap on two streams, each with its own workspace: all gradients are added
to those of the network, so they sum to what the two passes give one after the other.

The weights and biases of the two convolutions take one addition per pass of a sum that does not depend on
anything else, and two additions to zero commute: those are equal to the bit.  The output layer is summed with float
atomics of b blocks a pass in any order; 2 b additions round by 2^-24 of the running sum each, which is taken
to stay within 8 times the largest result.
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


@pytest.mark.parametrize("channels,n", [(16, 16), (16, 48), (32, 32)])
def test_backward_on_two_streams(cola, channels, n):
    print(f"lc overlap {channels} channels {n}^3", file=sys.stderr, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n)
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda")
    net = cola.LcNet(channels, in_scale=(0.5, 0.3, 0.3, 0.3), out_scale=0.4)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    passes = []
    for _ in streams:
        ws = cola.lc_workspace(n, channels, training=True)
        cola.lc_forward(net, rnd(n, n, n), rnd(3, n, n, n), ws, training=True)
        passes.append((ws, rnd(3, n, n, n)))
    net.grads.zero_()
    for ws, d_df in passes:
        cola.lc_backward(net, d_df, ws)
    want = net.grads.clone()
    conv = want.numel() - 3 * channels - 3  # the output layer comes last
    bound = 2 * (n ** 3 // 256) * 2.0 ** -24 * 8 * float(want[conv:].abs().max())
    for _ in range(20):
        net.grads.zero_()
        torch.cuda.synchronize()
        for s, (ws, d_df) in zip(streams, passes):
            with torch.cuda.stream(s):
                cola.lc_backward(net, d_df, ws)
        torch.cuda.synchronize()
        assert torch.equal(net.grads[:conv], want[:conv])
        assert float((net.grads[conv:] - want[conv:]).abs().max()) <= bound
