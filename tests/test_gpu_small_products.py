"""FP64 products of few tiles take a kernel of their own: bitwise the other kernel's results.

The kernel is chosen by the block's width too (for n > 512 up to 64 to 320 tiles of
128 x 64, by the length of the sum), and of the others those of up to 768 tiles take
narrower ones, so blocks on both sides of the lines must give every SNP the same bits; and for n <= 512, where it takes every width, the oracle decides.
Values are fractional, so that no SNP takes the integer product; unaligned
columns and sample counts off multiples of 16 read the block without a copy.
"""
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


def _study(n, p, m):
    Phi = synth.kinship(n, n)
    XL = synth.covariates(n, p, n, "gauss") if p > 1 else np.empty((n, 0))
    return Phi, XL, synth.phenotype(n, n), synth.genotypes(n, 0, m, n) * (1.0 / 3.0)


def _same(a, b, rows):
    for k in ("b", "sigma2", "v", "status"):
        assert np.array_equal(a[k][rows].view(np.uint8), b[k].view(np.uint8)), k


@pytest.mark.parametrize("precision,sweeps", [("fp64", 0), ("fp32_ir", 1)])
@pytest.mark.parametrize("n", [520, 768, 1009, 1024, 1025, 1700])
def test_both_sides_of_the_line(n, precision, sweeps):
    m = 64 * ((128 if n <= 1024 else 240) // -(-n // 128)) + 129   # one block above the line, its parts below
    Phi, XL, y, XR = _study(n, 4, m)
    ctx = GLSContext(_t(Phi), 0.4, _t(XL), _t(y), block_cols=m, precision=precision, refine_sweeps=sweeps)
    X = _t(XR)
    big = as_numpy(ctx.block(X))
    for j0, j1 in ((0, 1), (5, 22), (64, 700), (m - 9, m)):
        j1 = min(j1, m)
        _same(big, as_numpy(ctx.block(X[j0:j1])), slice(j0, j1))
    ctx.close()


@pytest.mark.parametrize("n,p", [(1025, 20), (1700, 4), (2309, 2), (2560, 1)])
def test_narrow_and_wide_tiles(n, p):
    """Above 768 tiles of 128 x 64, the wide tiles; the parts take the narrow ones or the kernel of few tiles."""
    m = 64 * (768 // -(-n // 128)) + 129
    Phi, XL, y, XR = _study(n, p, m)
    ctx = GLSContext(_t(Phi), 0.4, _t(XL) if p > 1 else None, _t(y), block_cols=m)
    X = _t(XR)
    big = as_numpy(ctx.block(X))
    for j0, j1 in ((3, 4), (64, 1100), (31, m - 1), (m - 700, m)):
        _same(big, as_numpy(ctx.block(X[j0:j1])), slice(j0, j1))
    ctx.close()


@pytest.mark.parametrize("n,p,m", [(5, 1, 7), (31, 4, 1), (128, 20, 33), (129, 3, 16), (255, 8, 15), (500, 4, 300), (512, 2, 130)])
def test_small_studies(n, p, m):
    Phi, XL, y, XR = _study(n, p, m)
    ctx = GLSContext(_t(Phi), 0.4, _t(XL) if p > 1 else None, _t(y), block_cols=m)
    got = as_numpy(ctx.block(_t(XR)))
    compare(got, O.gls_sequence(Phi, 0.4, XL, y, XR), 1e-10)
    off = torch.empty(m * n + 1, dtype=torch.float64, device=DEV)[1:].view(m, n)
    off.copy_(_t(XR))
    _same(got, as_numpy(ctx.block(off)), slice(0, m))
    _same(got, as_numpy(ctx.block(_t(XR[m // 2:]))), slice(m // 2, m))
    ctx.close()
