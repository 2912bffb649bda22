"""The eigensolver when its one-launch reduction gives up (needs an MI355X).

TUNE_EIG_POLLS = 1 makes a workgroup give up at the first word of another one that is
not there yet (every kernel still ends by itself); the matrix is then reduced
column by column, as with 0.  From the same Hermitian matrix both are the same
operations, so Rayleigh-Ritz and LOBPCG give the same bits; where a panel has gone before
(over 2048 columns) the restored lower triangle is the mirror of the upper one, equal
to rounding.  Against the default: eigenvalues to 2e-12 scale sqrt(M) (each
eigensolver's bound is 1e-12), orthonormality as for the other eigensolver sizes.
The smallest sizes, on both sides of the one that takes the one launch, against NumPy
with those bounds.
"""
import numpy as np
import pytest

import workloads as W
from paper_2604_11139_amd import binding as B

from gpu_util import system, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    B.lib()
    yield
    torch.cuda.synchronize()


def _close(ev, ref):
    assert np.abs(ev - ref).max() <= 2e-12 * np.abs(ref).max() * np.sqrt(ref.size)


@pytest.mark.parametrize("M", [64, 65, 96, 300, 777])
@pytest.mark.parametrize("lowprec", [False, True])
def test_rayleigh_ritz(M, lowprec):
    import torch
    with B.System(system("c1"), B.ABI_PREC_MIXED if lowprec else B.ABI_PREC_FP64) as g:
        X = to_dev(W.random_block(g.npw, M, 11)).to(torch.complex64 if lowprec
                                                    else torch.complex128)
        out = {}
        for polls in (g.get_tuning(B.TUNE_EIG_POLLS), 0, 1):
            g.set_tuning(B.TUNE_EIG_POLLS, polls)
            Y = X.clone()
            ev, _, _ = g.rayleigh_ritz(Y, lowprec=lowprec)
            out[polls] = (ev, to_host(Y))
        default, ev0, ev1 = out[2 ** 21], out[0], out[1]
        assert np.array_equal(ev0[0], ev1[0]) and np.array_equal(ev0[1], ev1[1])
        _close(ev1[0], default[0])
        G = ev1[1].astype(np.complex128)
        assert np.abs(G.conj().T @ G - np.eye(M)).max() <= (1e-4 if lowprec else 1e-11)


def test_lobpcg():
    with B.System(system("c1")) as g:
        X = to_dev(W.random_block(g.npw, 64, 12))
        out = []
        for polls in (0, 1):
            g.set_tuning(B.TUNE_EIG_POLLS, polls)
            Y = X.clone()
            ev, res, _ = g.lobpcg(Y, 2, 2)
            out.append((ev, res, to_host(Y)))
        for a, b in zip(*out):
            assert np.array_equal(a, b)


def test_after_a_panel():
    import torch
    M = 2100
    with B.System(W.make_system(2)) as g:
        gen = torch.Generator(device="cuda").manual_seed(5)
        X = torch.view_as_complex(torch.randn((M, g.npw, 2), generator=gen, device="cuda",
                                              dtype=torch.float64))
        ref, _, _ = g.rayleigh_ritz(X.clone())
        g.set_tuning(B.TUNE_EIG_POLLS, 1)
        Y = X.clone()
        ev, _, _ = g.rayleigh_ritz(Y)
        _close(ev, ref)
        G = Y.conj() @ Y.T.contiguous()
        assert float((G - torch.eye(M, device="cuda")).abs().max()) <= 1e-11


@pytest.mark.parametrize("m", [1, 2, 6, 7, 8, 9])
def test_smallest(m):
    import torch
    rng = np.random.default_rng(m)
    A = rng.standard_normal((m, m)) + 1j * rng.standard_normal((m, m))
    A = A + A.conj().T
    w, Z = (t.cpu().numpy() for t in B.zheev(torch.from_numpy(A).cuda()))
    ref = np.linalg.eigvalsh(A)
    scale = np.abs(ref).max()
    assert np.abs(w - ref).max() <= 1e-12 * scale * np.sqrt(m)
    assert np.abs(A @ Z - Z * w[None, :]).max() <= 1e-11 * scale
    assert np.abs(Z.conj().T @ Z - np.eye(m)).max() <= 1e-11


def test_parameter():
    with B.System(system("tiny_k")) as g:
        assert g.get_tuning(B.TUNE_EIG_POLLS) == 2 ** 21
        with pytest.raises(B.ChebfiError) as e:
            g.set_tuning(B.TUNE_EIG_POLLS, -1)
        assert e.value.code == B.ABI_ERR_ARG
