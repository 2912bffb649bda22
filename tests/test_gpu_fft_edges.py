"""Compile-time FFT passes at every edge they exist for, and on boxes that are
not cubes (needs an MI355X).

Square planes with an equal and with another z edge (z above 64 points included:
the occupied-plane mask then has two words), planes that are not square with a
listed and with an unlisted z edge, plane sizes that are no multiple of the z
passes' pencil count.  H X against the FP64 oracle to 1e-10 (FP64) and 2e-6
(mixed) per column; density to 1e-12 of its maximum (FP64) and 1e-6 (mixed); the
adjoint's three gradients to 1e-9 (FP64) and 1e-5 m (mixed) of their maxima: the
bounds of the same checks on the cubic boxes.
"""
import functools

import numpy as np
import pytest

import oracle as O
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


EDGES = [12, 15, 16, 18, 20, 24, 25, 27, 30, 32, 36, 40, 45, 48, 50, 54, 60, 64, 72, 75, 80, 81, 90,
         96]
# square planes: z longer and shorter; plane of another shape; unlisted edges (10, 9)
SLABS = [(20, 20, 75), (36, 36, 80), (54, 54, 25), (15, 15, 96), (25, 36, 72), (81, 12, 16),
         (20, 20, 10), (10, 10, 30), (9, 12, 10)]


@functools.lru_cache(maxsize=None)
def _system(ngrid):
    # the sphere just fits the shortest edge of the 8-bohr cell
    n = min(ngrid)
    gmax = min((n - 1) // 2 - 0.6, 6.0) * 2 * np.pi / 8.0
    s = W.make_system(310 + n, a=8.0, ecut=0.5 * gmax ** 2, n=n, natom=2, nband=5,
                      kpt_red=(0.2, 0.1, 0.3))
    s.ngrid = ngrid
    s.vloc = W.systems._gaussian_wells(s.tau, s.a, ngrid)
    return s


@functools.lru_cache(maxsize=None)
def _ham(ngrid):
    return O.Hamiltonian.from_system(_system(ngrid))


def _inputs(ngrid, mixed):
    import torch
    s, H = _system(ngrid), _ham(ngrid)
    X = W.random_block(H.npw, s.nband, s.tag)
    Wb = W.random_block(H.npw, s.nband, s.tag, stream=W.systems.WBLOCK)
    if mixed:
        X, Wb = (v.astype(np.complex64).astype(np.complex128) for v in (X, Wb))
    dt = torch.complex64 if mixed else torch.complex128
    return s, H, X, Wb, to_dev(X).to(dt), to_dev(Wb).to(dt)


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("ngrid", [(n, n, n) for n in EDGES] + SLABS)
def test_apply_H(ngrid, mixed):
    s, H, X, _, Xd, _ = _inputs(ngrid, mixed)
    with B.System(s, B.ABI_PREC_MIXED if mixed else B.ABI_PREC_FP64) as g:
        got = to_host(g.apply_H(Xd)).astype(np.complex128)
    assert col_rel_err(got, H(X)) <= (2e-6 if mixed else 1e-10)


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("ngrid", [(54, 54, 54), (36, 36, 80), (25, 36, 72), (20, 20, 10)])
def test_density_and_adjoint(ngrid, mixed):
    s, H, X, Wb, Xd, Wd = _inputs(ngrid, mixed)
    a, b, a0, m = 1.0, s.ecut + 1.0, -1.0, 3
    with B.System(s, B.ABI_PREC_MIXED if mixed else B.ABI_PREC_FP64) as g:
        rho = g.density(Xd).cpu().numpy()
        dV, dD, dX = g.filter_backward(Xd, Wd, m, a, b, a0, ckpt_every=2)
    ref = O.density(H, X)
    assert np.max(np.abs(rho - ref)) <= (1e-6 if mixed else 1e-12) * np.max(np.abs(ref))
    rV, rD, rX = O.filter_backward(H, X, Wb, m, a, b, a0)
    tol = 1e-5 * m if mixed else 1e-9
    for got, want in ((dV.cpu().numpy(), rV), (dD.cpu().numpy(), rD), (to_host(dX), rX)):
        assert np.max(np.abs(got.reshape(-1) - want.reshape(-1))) <= tol * np.max(np.abs(want))
