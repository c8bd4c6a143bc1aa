"""Low-precision products in small and large tiles: bitwise the same results on both sides of the line between them."""
import numpy as np
import pytest
import torch

from oracle import gls_oracle as O
from paper_1302_4332_amd import synth
from paper_1302_4332_amd.gls import GLSContext
from parity_util import as_numpy, compare

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _t(a):
    return torch.tensor(np.ascontiguousarray(a), device=DEV)


@pytest.mark.parametrize("precision,sweeps", [("fp32_ir", 1), ("fp16_ir", 2), ("bf16_ir", 3)])
@pytest.mark.parametrize("n", [1030, 1281])
def test_both_sides_of_the_line(n, precision, sweeps):
    m = 128 * (512 // -(-n // 256)) + 65   # one block above the line, its parts below
    Phi, XL, y = synth.kinship(n, n), synth.covariates(n, 4, n, "sex_age"), synth.phenotype(n, n)
    X = torch.randint(0, 3, (m, n), generator=torch.Generator(device=DEV).manual_seed(n), device=DEV).double()
    ctx = GLSContext(_t(Phi), 0.4, _t(XL), _t(y), block_cols=m, precision=precision, refine_sweeps=sweeps)
    big = as_numpy(ctx.block(X))
    for j0, j1 in ((0, 1), (63, 130), (m - 700, m)):
        part = as_numpy(ctx.block(X[j0:j1]))
        for k in ("b", "sigma2", "v", "status"):
            assert np.array_equal(big[k][j0:j1].view(np.uint8), part[k].view(np.uint8)), k
    ctx.close()


@pytest.mark.parametrize("n,m", [(3, 1), (64, 65), (257, 64), (513, 7)])
def test_small_studies(n, m):
    p = 1 if n == 3 else 4
    Phi, y = synth.kinship(n, n), synth.phenotype(n, n)
    XL = synth.covariates(n, 4, n, "sex_age") if p > 1 else np.empty((n, 0))
    XR = synth.genotypes(n, 0, m, n) + 0.125 * np.arange(n) / n
    for precision, sweeps in (("fp32_ir", 2), ("fp16_ir", 3), ("bf16_ir", 4)):
        ctx = GLSContext(_t(Phi), 0.4, _t(XL) if p > 1 else None, _t(y), block_cols=m, precision=precision,
                         refine_sweeps=sweeps)
        compare(as_numpy(ctx.block(_t(XR))), O.gls_sequence(Phi, 0.4, XL, y, XR), 1e-8)
        ctx.close()
