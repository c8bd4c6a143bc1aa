"""The factorization's widest nodes on the integer matrix cores (products by residues), against plain FP64.

From 2,304 rows and columns a node's products are formed modulo fifteen moduli.
n = 4,700 is the smallest that has such a node (37 blocks: 19 and 18 of 128, so
2,432 by 2,304), with ragged tiles and padding.  The whitened outputs are
compared with torch's FP64 Cholesky and triangular solves, for a matrix of
ordinary scale and for one whose rows and columns are scaled over 2^+-60 (the
factor's rows then are too, and the residues' own scaling has to follow).
The bar is the plain-FP64 one, 1e-10.
"""
import pytest
import torch

from paper_1302_4332_amd.gls import GLSContext

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("n,scaled", [(4700, False), (4865, True), (6001, False)])
def test_wide_nodes(n, scaled):
    g = torch.Generator(device=DEV).manual_seed(n)
    G = torch.randn(n, 1500, generator=g, device=DEV, dtype=torch.float64)
    M = (G @ G.T) / 1500 + 0.5 * torch.eye(n, dtype=torch.float64, device=DEV)
    y = torch.randn(n, generator=g, device=DEV, dtype=torch.float64)
    XL = torch.randn(n, 2, generator=g, device=DEV, dtype=torch.float64)
    XR = torch.randint(0, 3, (64, n), generator=g, device=DEV).double()
    L = torch.linalg.cholesky(M)

    def whitened(B):   # L^-1 B by blocks of rows
        out = torch.empty_like(B)
        for i in range(0, n, 1024):
            k = min(n, i + 1024)
            out[i:k] = torch.linalg.solve_triangular(L[i:k, i:k].contiguous(), B[i:k] - L[i:k, :i] @ out[:i], upper=False)
        return out

    A = torch.cat([whitened(XL), torch.zeros(n, 1, dtype=torch.float64, device=DEV)], 1)
    yt, Xt = whitened(y[:, None])[:, 0], whitened(XR.T.contiguous())
    if scaled:   # M -> S M S, X -> S X, y -> S y: the same coefficients
        s = 2.0 ** torch.randint(-60, 61, (n,), generator=g, device=DEV).double()
        M, y, XL, XR = s[:, None] * M * s, s * y, s[:, None] * XL, XR * s
    ctx = GLSContext(M.contiguous(), 1.0, XL.contiguous(), y, block_cols=64)
    b, s2, v, status = ctx.block(XR.contiguous())
    ctx.close()
    assert int(status.abs().sum()) == 0
    worst = 0.0
    for j in range(64):
        A[:, 2] = Xt[:, j]
        S = A.T @ A
        ref = torch.linalg.solve(S, A.T @ yt)
        worst = max(worst, float((b[j] - ref).abs().max() / ref.abs().max()))
        assert abs(float(v[j] / torch.linalg.inv(S)[2, 2]) - 1) <= 1e-10
    print(f"n={n} scaled={scaled}: {worst:.1e}")
    assert worst <= 1e-10


def test_pivot_inside_a_wide_node():
    """A pivot that fails in the right half of a wide node is reported as such: its trailing update came by residues."""
    n, pivot = 4700, 4400
    g = torch.Generator(device=DEV).manual_seed(5)
    G = torch.randn(n, 64, generator=g, device=DEV, dtype=torch.float64)
    M = (G @ G.T) / 64 + torch.eye(n, dtype=torch.float64, device=DEV)
    M[pivot - 1, pivot - 1] = -1.0
    from paper_1302_4332_amd.gls import GLSError
    with pytest.raises(GLSError) as e:
        GLSContext(M.contiguous(), 1.0, None, torch.ones(n, dtype=torch.float64, device=DEV), block_cols=4)
    assert e.value.status == -2 and e.value.info == pivot
