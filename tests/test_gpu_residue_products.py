"""The factorization's widest nodes on the integer matrix cores (products by residues), against plain FP64.

From 2,304 rows and columns a node's products are formed modulo sixteen moduli.
n = 4,700 is the smallest that has such a node (37 blocks: 19 and 18 of 128, so
2,432 by 2,304), with ragged tiles and padding.  The whitened outputs are
compared with torch's FP64 Cholesky and triangular solves, for a matrix of
ordinary scale and for one whose rows and columns are scaled over 2^+-60 (the
factor's rows then are too, and the residues' own scaling has to follow).
The bar is the plain-FP64 one, 1e-10.
"""
import numpy as np
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


def _pieces(A, count):
    """A as `count` matrices of 17-bit integers times a power of two each (relative to A's largest entry), whose products
    over up to 2^19 terms are exact in FP64."""
    if not A.any():
        return [A] * count
    out, scale = [], 2.0 ** torch.ceil(torch.log2(A.abs().max())).item()
    R = A.clone()
    for _ in range(count):
        scale *= 2.0 ** -17
        P = torch.round(R / scale) * scale
        out.append(P)
        R = R - P
    return out


def _exact_product(A, B):
    """A B to far below FP64's precision, as a longdouble array: every partial product is exact."""
    out = np.zeros((A.shape[0], B.shape[1]), dtype=np.longdouble)
    Ap, Bp = _pieces(A, 5), _pieces(B, 5)
    for i in range(5):
        for j in range(5 - i):
            out += (Ap[i] @ Bp[j]).cpu().numpy()
    return out


def _inverse_factor(A, leaves):
    """Cholesky factor's inverse of the lower triangle of A by the same recursion over blocks of 128 rows, every product
    torch's FP64 one."""
    n = A.shape[0]
    if leaves == 1:
        L = torch.linalg.cholesky(A)
        return torch.linalg.solve_triangular(L, torch.eye(n, dtype=A.dtype, device=A.device), upper=False)
    h = leaves // 2 * 128
    I11 = _inverse_factor(A[:h, :h].contiguous(), leaves // 2)
    L21 = A[h:, :h] @ I11.T.contiguous()
    I22 = _inverse_factor(A[h:, h:] - L21 @ L21.T.contiguous(), leaves - leaves // 2)
    out = torch.zeros_like(A)
    out[:h, :h], out[h:, h:] = I11, I22
    out[h:, :h] = -(I22 @ (L21 @ I11))
    return out


@pytest.mark.parametrize("n", [4700, 6001])
def test_near_singular(n):
    """h2 near 1 and samples in nearly equal pairs (M's condition is about 1e7): the coefficients' error against refined
    solves (rms over 64 SNPs) is within twice that of the same factorization with every product in FP64.  (Both apply an
    explicit inverse, whose error is several times that of triangular solves here.)"""
    g = torch.Generator(device=DEV).manual_seed(n)
    dd = dict(generator=g, device=DEV, dtype=torch.float64)
    G = torch.randn(n, 3000, **dd)
    h = n // 2
    G[h:2 * h] = G[:h] + 1e-3 * torch.randn(h, 3000, **dd)
    Phi = (G @ G.T) / 3000
    Phi = 0.5 * (Phi + Phi.T)
    h2 = 1.0 - 2.0 ** -20
    y, XL = torch.randn(n, **dd), torch.randn(n, 2, **dd)
    XR = torch.randint(0, 3, (64, n), generator=g, device=DEV).double() * (1.0 / 3.0)   # not whole: the FP64 product
    ctx = GLSContext(Phi.contiguous(), h2, XL.contiguous(), y, block_cols=64)
    b, _, _, status = ctx.block(XR.contiguous())
    ctx.close()
    assert int(status.abs().sum()) == 0
    M = h2 * Phi + (1.0 - h2) * torch.eye(n, dtype=torch.float64, device=DEV)
    L = torch.linalg.cholesky(M)
    V = torch.cat([XL, y[:, None], XR.T], 1).contiguous()
    Zl = torch.cholesky_solve(V, L).cpu().numpy().astype(np.longdouble)
    for _ in range(4):   # each step gains the digits that the condition leaves of FP64's sixteen
        lo = torch.tensor((Zl - Zl.astype(np.float64)).astype(np.float64), device=DEV)
        hi = torch.tensor(Zl.astype(np.float64), device=DEV)
        R = V.cpu().numpy().astype(np.longdouble) - _exact_product(M, hi) - _exact_product(M, lo)
        Zl = Zl + torch.cholesky_solve(torch.tensor(R.astype(np.float64), device=DEV), L).cpu().numpy()

    def coefficients(A, B):
        S, out = A.T @ B, []
        for j in range(64):
            at = [0, 1, 3 + j]
            T, r = S[np.ix_(at, at)], S[at, 2]
            x = np.linalg.solve(T.astype(np.float64), r.astype(np.float64)).astype(np.longdouble)
            for _ in range(2):
                x = x + np.linalg.solve(T.astype(np.float64), (r - T @ x).astype(np.float64))
            out.append(x)
        return np.array(out)

    W = (_inverse_factor(M, -(-n // 128)) @ V).cpu().numpy().astype(np.longdouble)
    ref, f64 = coefficients(V.cpu().numpy().astype(np.longdouble), Zl), coefficients(W, W)
    rms = lambda x: float(np.sqrt(np.mean((np.abs(x - ref).max(1) / np.abs(ref).max(1)) ** 2)))
    mine, theirs = rms(b.cpu().numpy().astype(np.longdouble)), rms(f64)
    print(f"n={n}: {mine:.1e} against {theirs:.1e}")
    assert mine <= 2.0 * theirs


@pytest.mark.parametrize("n,scaled", [(4700, False), (9100, True)])
def test_room_for_fewer_columns(n, scaled):
    """Handles of small blocks form the products some 192 k columns at a time, those of large ones at once: the same
    integers, so the same factor and the same results, bit for bit.  (9,100 samples have wide nodes at two depths.)"""
    g = torch.Generator(device=DEV).manual_seed(n)
    G = torch.randn(n, 600, generator=g, device=DEV, dtype=torch.float64)
    M = (G @ G.T) / 600 + 0.5 * torch.eye(n, dtype=torch.float64, device=DEV)
    if scaled:
        s = 2.0 ** torch.randint(-9, 10, (n,), generator=g, device=DEV).double()
        M = s[:, None] * M * s
    y = torch.randn(n, generator=g, device=DEV, dtype=torch.float64)
    XR = torch.randn(8, n, generator=g, device=DEV, dtype=torch.float64)
    outs = []
    for bc in (8, 8192):
        ctx = GLSContext(M.contiguous(), 1.0, None, y, block_cols=bc)
        outs.append([t.cpu().numpy().copy() for t in ctx.block(XR)])
        ctx.close()
    for a, b in zip(*outs):
        assert np.array_equal(a.view(np.uint8), b.view(np.uint8))
