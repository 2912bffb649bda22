"""The batched filter over many boxes at once (needs an MI355X).

One batch of cubic boxes of edges from 12 to 96 (even, odd, below and above 64
points, several systems of one edge with uneven band counts) and boxes without
compile-time passes (edge 10, 12 x 15 x 16), and one of 70 systems, more than a
wave finds in one step, of which all but two share an edge.  Each system's block
against the single-system filter of the same handle: 1e-12 (FP64), 1e-5 m (mixed:
two mixed filters, each within 5e-6 m of FP64), overlapped and in line, replayed
and eager.
"""
import numpy as np
import pytest

import workloads as W
from paper_2604_11139_amd import binding as B

from gpu_util import col_rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    B.lib()
    yield
    torch.cuda.synchronize()


def _system(i, n, nband, natom=2):
    s = W.make_system(350 + i, a=8.0, ecut=min(0.5 * ((n - 1) // 2 - 0.6) ** 2 * 0.617, 9.0), n=n,
                      natom=natom, nband=nband, kpt_red=(0.2, 0.1, 0.3))
    return s


def _edges():
    out = [_system(i, n, nb, 1 + i % 3)
           for i, (n, nb) in enumerate([(12, 3), (18, 7), (45, 2), (45, 5), (50, 3), (64, 2),
                                        (72, 3), (96, 2), (10, 4), (36, 33)])]
    s = _system(20, 12, 5)
    s.ngrid = (12, 15, 16)
    s.vloc = W.systems._gaussian_wells(s.tau, s.a, s.ngrid)
    return out + [s]


def _many():
    return [_system(30 + i, 15 if i in (0, 69) else 12, 1 + i % 4, 1) for i in range(70)]


@pytest.mark.parametrize("graph,overlap", [(True, True), (False, False)])
@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("which", ["edges", "many"])
def test_batch_against_single(which, mixed, graph, overlap):
    import torch
    systems = _edges() if which == "edges" else _many()
    m = 3
    with B.Batch(systems, B.ABI_PREC_MIXED if mixed else B.ABI_PREC_FP64) as batch:
        batch.use_graph(graph)
        batch.use_overlap(overlap)
        dt = torch.complex64 if mixed else torch.complex128
        Xs = [to_dev(W.random_block(h.npw, s.nband, s.tag)).to(dt)
              for h, s in zip(batch.systems, systems)]
        bounds = [(1.0, s.ecut + 1.0, -1.0) for s in systems]
        for _ in range(2):
            out = batch.cheb_filter(Xs, m, bounds)
        for h, s, X, Y, bd in zip(batch.systems, systems, Xs, out, bounds):
            ref = to_host(h.cheb_filter(X, m, *bd)).astype(np.complex128)
            assert col_rel_err(to_host(Y).astype(np.complex128), ref) <= (
                1e-5 * m if mixed else 1e-12), (s.ngrid, s.nband)
