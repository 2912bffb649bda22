"""The split-BF16 Gram products of more than one output tile (needs an MI355X).

Only the 128 x 128 tiles on and above the diagonal are multiplied and the rest
is mirrored: band counts below, at and above one and two tiles and not a multiple
of the 32 x 32 blocks of the sum.  The Ritz values of the split-BF16 Rayleigh-Ritz
against the oracle's on the same complex64 block, 1e-4 max|lambda| (the bound of
the one-pass form), Ritz vectors orthonormal to 1e-4, and the FP64 form of the
same block to 1e-8.
"""
import numpy as np
import pytest

import oracle as O
import workloads as W
from paper_2604_11139_amd import binding as B

from gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    B.lib()
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("nband", [1, 31, 127, 128, 129, 200, 257])
def test_rayleigh_ritz(nband):
    import torch
    s = W.make_system(340, a=14.0, ecut=8.0, n=36, natom=6, nband=nband, kpt_red=(0.1, 0.2, 0.3))
    H = O.Hamiltonian.from_system(s)
    X = W.random_block(H.npw, nband, s.tag)
    # columns concentrated on the low plane waves, as a filter leaves them
    Y = X / (1.0 + H.sphere.kinetic[:, None] ** 2)
    Y = Y / np.linalg.norm(Y, axis=0)[None, :]
    Y = Y.astype(np.complex64).astype(np.complex128)
    ref = O.rayleigh_ritz(H, Y)["eval"]
    with B.System(s, precision=B.ABI_PREC_MIXED) as g:
        Yd = to_dev(Y).to(torch.complex64)
        Y64 = Yd.clone()
        ev, _, flags = g.rayleigh_ritz(Yd, lowprec=True)
        Psi = to_host(Yd).astype(np.complex128)
        ev64, _, _ = g.rayleigh_ritz(Y64)
    assert flags & B.RR_LOWPREC
    scale = np.abs(ref).max()
    assert np.abs(ev - ref).max() <= 1e-4 * scale
    assert np.abs(Psi.conj().T @ Psi - np.eye(nband)).max() <= 1e-4
    assert np.abs(ev64 - ref).max() <= 1e-8
