"""The factorization's small nodes: one 128-row block, its panels of 16, and the first levels above it.

Sample counts at the edges of a panel, of a block and of nodes of unequal
halves, against the CPU oracle at the plain-FP64 bar; and the failing pivot of
matrices that are not positive definite, at the edges of the panels and blocks.
"""
import numpy as np
import pytest
import torch

from oracle import gls_oracle as O
from paper_1302_4332_amd import synth
from paper_1302_4332_amd.gls import GLSContext, GLSError
from parity_util import as_numpy, compare

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _t(a):
    return torch.tensor(np.ascontiguousarray(a), device=DEV)


@pytest.mark.parametrize("n", [3, 16, 17, 113, 127, 128, 129, 257, 385, 640, 897, 1153])
@pytest.mark.parametrize("h2", [0.3, 0.9])
def test_sizes(n, h2):
    p = 1 if n == 3 else 2
    Phi, XL, y = synth.kinship(n, n), synth.covariates(n, p, n, "gauss"), synth.phenotype(n, n)
    XR = synth.genotypes(n, 0, 40, n) + 0.125 * np.arange(n) / n   # no whole numbers, no constant column
    ctx = GLSContext(_t(Phi), h2, _t(XL) if p > 1 else None, _t(y), block_cols=40)
    err = compare(as_numpy(ctx.block(_t(XR))), O.gls_sequence(Phi, h2, XL, y, XR), 1e-10)
    ctx.close()
    print(f"n={n} h2={h2}: {err:.1e}")


@pytest.mark.parametrize("pivot", [1, 2, 16, 17, 64, 112, 113, 128, 129, 256, 257, 300])
def test_failing_pivot(pivot):
    n = 300
    rng = np.random.default_rng(pivot)
    G = rng.standard_normal((n, n)) / np.sqrt(n)
    A = G @ G.T + np.eye(n)
    A[pivot - 1, pivot - 1] = -1.0   # every leading minor before it is positive
    with pytest.raises(GLSError) as e:
        GLSContext(_t(A), 1.0, None, _t(rng.standard_normal(n)), block_cols=4)
    assert e.value.status == -2 and e.value.info == pivot
