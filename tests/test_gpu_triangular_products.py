"""Products with a triangular factor in the Rayleigh-Ritz step (needs an MI355X).

The rotation by the inverse Cholesky factor of the two-pass split-BF16 form, band
counts below, at and above one and two 128-column tiles, and the FP64 reductions
above the band count from which they leave out the zero half (64 x 64 tiles in more
than two rounds; 712 and 720: a remainder of 8 and 16 past a multiple of 64).
Against the oracle on the same block: Ritz values to 1e-4 max|lambda| and Ritz
vectors orthonormal to 1e-4 (split-BF16), 1e-8 and 1e-10 (FP64), the bounds of the
same checks of the other forms.
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


def _case(nband, ecut):
    """A block whose neighbouring columns overlap (pivots^2 of its equilibrated Gram
    matrix near 1 / 2.6)."""
    s = W.make_system(350, a=14.0, ecut=ecut, n=40, natom=4, nband=nband, kpt_red=(0.1, 0.2, 0.3))
    H = O.Hamiltonian.from_system(s)
    X = W.random_block(H.npw, nband + 2, s.tag) / (1.0 + H.sphere.kinetic[:, None])
    X = X / np.linalg.norm(X, axis=0)[None, :]
    Y = X[:, 2:] + 0.9 * X[:, 1:-1] + 0.9 * X[:, :-2]
    Y = Y / np.linalg.norm(Y, axis=0)[None, :]
    Y = Y.astype(np.complex64).astype(np.complex128)
    return s, Y, O.rayleigh_ritz(H, Y)["eval"]


@pytest.mark.parametrize("nband", [1, 33, 128, 129, 255, 257])
def test_two_pass_rotation(nband):
    import torch
    s, Y, ref = _case(nband, 8.0)
    with B.System(s, precision=B.ABI_PREC_MIXED) as g:
        Yd = to_dev(Y).to(torch.complex64)
        ev, _, flags = g.rayleigh_ritz(Yd, lowprec=True)
        Psi = to_host(Yd).astype(np.complex128)
    assert flags == (B.RR_LOWPREC | B.RR_TWO_PASS if nband > 2 else B.RR_LOWPREC)
    assert np.abs(ev - ref).max() <= 1e-4 * np.abs(ref).max()
    assert np.abs(Psi.conj().T @ Psi - np.eye(nband)).max() <= 1e-4


@pytest.mark.parametrize("nband", [640, 712, 720])
def test_fp64_reduction(nband):
    s, Y, ref = _case(nband, 10.0)
    with B.System(s) as g:
        Yd = to_dev(Y)
        ev, _, _ = g.rayleigh_ritz(Yd)
        Psi = to_host(Yd)
    assert np.abs(ev - ref).max() <= 1e-8
    assert np.abs(Psi.conj().T @ Psi - np.eye(nband)).max() <= 1e-10
