"""Cholesky at the ends of its range (needs an MI355X).

A matrix scaled down by a power of two until its entries are denormal: the factor is
the unscaled one's, to what the rounding of the entries (2^-1074) leaves, 2^-46 here; each
of the m updates of an entry rounds once more, and with eigenvalues in [1, 2] the
factor passes that on: 4 m 2^-46.
An ill-conditioned one (1e11): the backward error |U^H U - A|_F against the bound of a
stable factorisation, (m + 1) eps trace(A), with a factor of 8 for complex arithmetic
and the product with the diagonal blocks' inverses.
Rayleigh-Ritz of a block whose Gram matrix has condition 1e8: orthonormal to
8 m eps 1e8 (one Cholesky orthonormalisation, the triangular inverse by doubling).
"""
import numpy as np
import pytest

import workloads as W
from paper_2604_11139_amd import binding as B

from gpu_util import system, to_dev, to_host

pytestmark = pytest.mark.gpu
EPS = np.finfo(float).eps


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    B.lib()
    yield
    torch.cuda.synchronize()


def _unitary(m, seed):
    rng = np.random.default_rng([m, seed])
    return np.linalg.qr(rng.standard_normal((m, m)) + 1j * rng.standard_normal((m, m)))[0]


def _hpd(m, eigs):
    Q = _unitary(m, 1)
    A = (Q * eigs) @ Q.conj().T
    return (A + A.conj().T) / 2


def _factor(A):
    import torch
    return np.triu(B.zpotrf_upper(torch.from_numpy(A).cuda()).cpu().numpy())


@pytest.mark.parametrize("m", [31, 32, 33, 64, 97])
def test_denormal(m):
    A = _hpd(m, np.linspace(1.0, 2.0, m))
    small = A * 2.0 ** -514 * 2.0 ** -514
    U = _factor(small) * 2.0 ** 514
    ref = np.linalg.cholesky(A).conj().T
    assert np.abs(U - ref).max() <= 4 * m * 2.0 ** -46


@pytest.mark.parametrize("m", [33, 64, 200, 513])
def test_ill_conditioned(m):
    A = _hpd(m, np.logspace(-11, 0, m))
    U = _factor(A)
    assert np.linalg.norm(U.conj().T @ U - A) <= 8 * (m + 1) * EPS * np.trace(A).real


@pytest.mark.parametrize("m", [33, 96, 200])
def test_rayleigh_ritz_ill_conditioned(m):
    with B.System(system("c1")) as g:
        Q = np.linalg.qr(W.random_block(g.npw, m, 5))[0]
        X = (Q * np.logspace(-4, 0, m)) @ _unitary(m, 2)
        Y = to_dev(X)
        g.rayleigh_ritz(Y)
        P = to_host(Y)
        assert np.abs(P.conj().T @ P - np.eye(m)).max() <= 8 * m * EPS * 1e8
