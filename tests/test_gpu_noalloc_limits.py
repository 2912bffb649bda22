"""No-allocation H applications just below the scratch array's limit (needs an MI355X).

Sizes whose work buffers fit the 64 MiB with the fewest K chunks of the projection but
not with the chunk count a call with room takes.
140 bands of 22119 plane waves and 256 projectors on a planes projection: the block's
bf16 planes (25 MB) and the projector part E (25 MB) leave 17 MB for partial products,
and 64 chunks would take 18.
255 bands of 1503 plane waves on the comparison forms of the mixed products: the boxes,
made before the products, would leave 0.25 MB of the array.
Against abi_apply_H at the no-allocation tests' mixed bar (2e-6 per column).
"""
import numpy as np
import pytest

import workloads as W
from paper_2604_11139_amd import binding as B

from gpu_util import col_rel_err, system, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    B.lib()
    yield
    torch.cuda.synchronize()


def _against_apply(g, nband):
    import torch
    X = torch.from_numpy(W.random_block(g.npw, nband, 43).T.copy()).to("cuda").to(torch.complex64)
    ref = g.apply_H(X)
    out = torch.full_like(X, float("nan"))
    g.apply_H_noalloc(X, out)
    torch.cuda.synchronize()
    got, want = (to_host(t).astype(np.complex128) for t in (out, ref))
    assert np.isfinite(got).all()
    assert col_rel_err(got, want) <= 2e-6


@pytest.mark.parametrize("proj", [0, 7])
def test_planes_projection(proj):
    with B.System(W.make_system(2), precision=B.ABI_PREC_MIXED) as g:
        g.set_tuning(B.TUNE_PROJ, proj)
        _against_apply(g, 140)


@pytest.mark.parametrize("form", [1, 2])
def test_products_after_the_boxes(form):
    with B.System(system("c1"), precision=B.ABI_PREC_MIXED) as g:
        g.set_tuning(B.TUNE_MIXED_GEMM, form)
        _against_apply(g, 255)
