"""Real-space sums over bands (density, potential gradient of the adjoint) formed in
the z pass (needs an MI355X).

Every edge with compile-time transforms at a band count below one band per
workgroup, and two edges at band counts that give each workgroup several bands with
a remainder.  Density against the FP64 oracle to 1e-12 of its maximum (FP64) and
1e-6 (mixed); the adjoint's three gradients to 1e-9 (FP64) and 1e-5 m (mixed) of
their maxima: the bounds of the same checks elsewhere.  The gradients do not depend
on the checkpoint interval (bitwise).
"""
import functools

import numpy as np
import pytest

import oracle as O
import workloads as W
from paper_2604_11139_amd import binding as B

from gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu

EDGES = [12, 15, 16, 18, 20, 24, 25, 27, 30, 32, 36, 40, 45, 48, 50, 54, 60, 64, 72, 75, 80, 81, 90,
         96]


@functools.lru_cache(maxsize=None)
def _case(n, nband):
    gmax = min((n - 1) // 2 - 0.6, 4.0) * 2 * np.pi / 8.0
    s = W.make_system(710 + n, a=8.0, ecut=0.5 * gmax ** 2, n=n, natom=1, nband=nband,
                      kpt_red=(0.1, 0.2, 0.4))
    return s, O.Hamiltonian.from_system(s)


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("n,nband", [(n, 3) for n in EDGES] + [(27, 205), (36, 155)])
def test_sums_over_bands(n, nband, mixed):
    import torch
    s, H = _case(n, nband)
    X = W.random_block(H.npw, nband, s.tag)
    Wb = W.random_block(H.npw, nband, s.tag, stream=W.systems.WBLOCK)
    if mixed:
        X, Wb = (v.astype(np.complex64).astype(np.complex128) for v in (X, Wb))
    dt = torch.complex64 if mixed else torch.complex128
    Xd, Wd = to_dev(X).to(dt), to_dev(Wb).to(dt)
    w = 0.25 + np.arange(nband) % 7
    a, b, a0, m = 1.0, s.ecut + 1.0, -1.0, 2
    with B.System(s, B.ABI_PREC_MIXED if mixed else B.ABI_PREC_FP64) as g:
        rho = g.density(Xd, w)
        twice = g.density_add(Xd, rho.clone(), w).cpu().numpy()
        rho = rho.cpu().numpy()
        grads = [t.cpu() for t in g.filter_backward(Xd, Wd, m, a, b, a0)]
        again = [t.cpu() for t in g.filter_backward(Xd, Wd, m, a, b, a0, ckpt_every=1)]
    ref = O.density(H, X, w)
    assert np.max(np.abs(rho - ref)) <= (1e-6 if mixed else 1e-12) * np.max(np.abs(ref))
    assert np.max(np.abs(twice - 2 * ref)) <= (2e-6 if mixed else 2e-12) * np.max(np.abs(ref))
    assert all(torch.equal(x, y) for x, y in zip(grads, again))
    refs = O.filter_backward(H, X, Wb, m, a, b, a0)
    tol = 1e-5 * m if mixed else 1e-9
    for i, (got, want) in enumerate(zip(grads, refs)):
        got = to_host(got) if i == 2 else got.numpy()
        assert np.max(np.abs(got.reshape(-1) - want.reshape(-1))) <= tol * np.max(np.abs(want))
