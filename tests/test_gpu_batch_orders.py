"""The batched filter's launch orders over many boxes (needs an MI355X).

Eager launches with the projector products on the second stream, joined before the first
edge's last pass, against the same launches in line: the same bits, over batches of many
edges, of boxes without compile-time passes alone and among others, and of 70 systems.
The autotuner leaves the chosen order alone.
"""
import pytest

import workloads as W
from paper_2604_11139_amd import binding as B

from gpu_util import to_dev
from test_gpu_batch_edges import _edges, _many, _system

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    B.lib()
    yield
    torch.cuda.synchronize()


def _blocks(batch, systems, dt):
    return [to_dev(W.random_block(h.npw, s.nband, s.tag)).to(dt)
            for h, s in zip(batch.systems, systems)]


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("which", ["edges", "many", "runtime"])
def test_eager_overlap(which, mixed):
    import torch
    systems = {"edges": _edges, "many": _many,
               "runtime": lambda: [_system(20 + i, 10, 4 + 5 * i) for i in range(3)]}[which]()
    bounds = [(1.0, s.ecut + 1.0, -1.0) for s in systems]
    with B.Batch(systems, B.ABI_PREC_MIXED if mixed else B.ABI_PREC_FP64) as batch:
        batch.use_graph(False)
        Xs = _blocks(batch, systems, torch.complex64 if mixed else torch.complex128)
        batch.use_overlap(False)
        ref = [Y.clone() for Y in batch.cheb_filter(Xs, 4, bounds)]
        batch.use_overlap(True)
        for rep in range(3):
            out = batch.cheb_filter(Xs, 4, bounds)
            torch.cuda.synchronize()
            for s, Y, R in zip(systems, out, ref):
                assert torch.equal(Y, R), (s.ngrid, s.nband, rep)


@pytest.mark.parametrize("graph", [False, True])
def test_autotune_in_either_order(graph):
    import torch
    systems = _edges()[:4]
    bounds = [(1.0, s.ecut + 1.0, -1.0) for s in systems]
    with B.Batch(systems, B.ABI_PREC_MIXED) as batch:
        batch.use_graph(graph)
        batch.use_overlap(True)
        Xs = _blocks(batch, systems, torch.complex64)
        ref = [Y.clone() for Y in batch.cheb_filter(Xs, 4, bounds)]
        batch.autotune(Xs, 4, bounds)
        out = batch.cheb_filter(Xs, 4, bounds)
        torch.cuda.synchronize()
        for s, Y, R in zip(systems, out, ref):  # cubic listed edges: one form of the passes
            assert torch.equal(Y, R), (s.ngrid, s.nband)
