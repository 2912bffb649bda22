"""Calls that only wait for the caller's stream (needs an MI355X).

With a kernel of some tenths of a second on the default stream, a Rayleigh-Ritz (FP64) or
LOBPCG pass on a stream of its own returns while that kernel still runs.  The first
calls (they allocate, which waits for the device) are made before.  Streams can share
a hardware queue, which makes one wait for the other whatever the library does: a
stream is taken on which a small copy gets past the busy one.
"""
import pytest

import workloads as W
from paper_2604_11139_amd import binding as B

from gpu_util import system, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    B.lib()
    yield
    torch.cuda.synchronize()


def _busy():
    """An event behind a spinning kernel (one wave) on the default stream."""
    import torch
    with torch.cuda.stream(torch.cuda.default_stream()):
        torch.cuda._sleep(int(5e8))
        e = torch.cuda.Event()
        e.record()
    return e


def _free_stream():
    """A stream that runs beside the default one, or None."""
    import torch
    x = torch.zeros(64, device="cuda")
    for _ in range(8):
        s = torch.cuda.Stream()
        torch.cuda.synchronize()
        e = _busy()
        with torch.cuda.stream(s):
            y = x.clone()
            s.synchronize()
        free = not e.query()
        torch.cuda.synchronize()
        del y
        if free:
            return s
    return None


@pytest.mark.parametrize("call", ["rayleigh_ritz", "lobpcg"])
def test_default_stream_is_left_alone(call):
    import torch
    st = _free_stream()
    if st is None:
        pytest.skip("every stream shares the default stream's hardware queue")
    s = system("c1")
    with torch.cuda.stream(st), B.System(s) as g:
        X = to_dev(W.random_block(g.npw, 32, 7))
        Y = X.clone()

        def run():
            Y.copy_(X)
            if call == "rayleigh_ritz":
                return g.rayleigh_ritz(Y)[0]
            return g.lobpcg(Y, 1, 1)[0]

        first = run()
        torch.cuda.synchronize()
        busy = _busy()
        again = run()
        still = not busy.query()
        torch.cuda.synchronize()
    assert still, "the call waited for the default stream"
    assert (first == again).all()
