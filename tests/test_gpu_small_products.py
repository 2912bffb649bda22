"""Projector products of blocks too small to fill the chip (needs an MI355X).

One to nine atoms and one to 130 bands: a single output tile and several, one
K chunk per few K steps, chunk counts below and above the one from which several
waves share a row's partials, and band counts around the 64 of a workgroup.  H X
and a degree-2 filter against the FP64 oracle with a nonlocal part scaled up to
the size of the local one, 1e-10 / 1e-9 (FP64) and 2e-6 / 1e-5 (mixed) per
column; the no-allocation call against the same oracle.
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


@functools.lru_cache(maxsize=None)
def _ham(natom):
    s = W.make_system(330 + natom, a=10.0, ecut=6.0, n=25, natom=natom, nband=130,
                      kpt_red=(0.1, 0.0, 0.2), d_scale=20.0)
    return s, O.Hamiltonian.from_system(s)


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("nband", [1, 2, 15, 63, 64, 65, 130])
@pytest.mark.parametrize("natom", [1, 2, 9])
def test_small_products(natom, nband, mixed):
    import torch
    s, H = _ham(natom)
    X = W.random_block(H.npw, nband, s.tag)
    if mixed:
        X = X.astype(np.complex64).astype(np.complex128)
    Xd = to_dev(X).to(torch.complex64 if mixed else torch.complex128)
    a, b, a0 = 1.0, s.ecut + 2.0, -2.0
    with B.System(s, B.ABI_PREC_MIXED if mixed else B.ABI_PREC_FP64) as g:
        got = to_host(g.apply_H(Xd)).astype(np.complex128)
        na = torch.full_like(Xd, float("nan"))
        g.apply_H_noalloc(Xd, na)
        Y = to_host(g.cheb_filter(Xd, 2, a, b, a0)).astype(np.complex128)
    ref = H(X)
    assert col_rel_err(got, ref) <= (2e-6 if mixed else 1e-10)
    assert col_rel_err(to_host(na).astype(np.complex128), ref) <= (2e-6 if mixed else 1e-10)
    assert col_rel_err(Y, O.cheb_filter(H, X, 2, a, b, a0)) <= (1e-5 if mixed else 1e-9)
