"""The register-resident tridiagonalisation at its edges (needs an MI355X).

Sizes around its workgroups' columns (8 per workgroup), its threads' rows (512,
1024, 2048) and its limit (2049 starts with a panel of the blocked form);
matrices whose reflectors are trivial (diagonal, real tridiagonal) and a
block diagonal one, whose columns vanish below a block in mid-reduction.
Bounds as for the other eigensolver sizes: eigenvalues to 1e-12 scale sqrt(m),
residual and orthonormality to 1e-11.  Two threads on two streams at once, each
against its own matrix.
"""
import threading

import numpy as np
import pytest

from paper_2604_11139_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    B.lib()
    yield
    torch.cuda.synchronize()


def _random(m, seed=0):
    rng = np.random.default_rng([m, seed])
    A = rng.standard_normal((m, m)) + 1j * rng.standard_normal((m, m))
    return A + A.conj().T


def _check(A, w, Z):
    m = A.shape[0]
    w, Z = w.cpu().numpy(), Z.cpu().numpy()
    ref = np.linalg.eigvalsh(A)
    scale = max(np.abs(ref).max(), 1e-300)
    assert np.all(np.diff(w) >= 0)
    assert np.abs(w - ref).max() <= 1e-12 * scale * np.sqrt(m)
    assert np.abs(A @ Z - Z * w[None, :]).max() <= 1e-11 * scale
    assert np.abs(Z.conj().T @ Z - np.eye(m)).max() <= 1e-11


@pytest.mark.parametrize("m", [2, 3, 8, 9, 16, 17, 511, 512, 513, 1023, 1024, 1025, 2047, 2049])
def test_sizes(m):
    import torch
    A = _random(m)
    _check(A, *B.zheev(torch.from_numpy(A).cuda()))


@pytest.mark.parametrize("kind", ["diagonal", "tridiagonal", "blocks"])
def test_trivial_reflectors(kind):
    import torch
    m = 150
    rng = np.random.default_rng(5)
    if kind == "blocks":
        A = np.zeros((m, m), dtype=np.complex128)
        A[:60, :60], A[60:, 60:] = _random(60), _random(90)
    else:
        A = np.diag(rng.standard_normal(m)).astype(np.complex128)
        if kind == "tridiagonal":
            e = rng.standard_normal(m - 1)
            A += np.diag(e, 1) + np.diag(e, -1)
    _check(A, *B.zheev(torch.from_numpy(A).cuda()))


def test_two_streams():
    import torch
    mats = [_random(700, s) for s in (1, 2)]
    out = [None, None]

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            a = torch.from_numpy(mats[i]).cuda()
            for _ in range(3):
                out[i] = B.zheev(a)
            torch.cuda.current_stream().synchronize()

    ts = [threading.Thread(target=work, args=(i,)) for i in (0, 1)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for A, (w, Z) in zip(mats, out):
        _check(A, w, Z)
