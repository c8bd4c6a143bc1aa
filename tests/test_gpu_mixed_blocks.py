"""Blocks of many SNPs, whole-number and fractional ones mixed: each product forms its own columns.

Such blocks run on the kernels of many tiles (160 SNPs of the integer product, 64
or 32 of the FP64 one), which take their columns by lists.  Small blocks run on the
kernels of few tiles, which find theirs by flags in place; both give every SNP the
same bits, so that a large block can be checked against small ones.  Some SNPs are
also held to the CPU oracle at the plain-FP64 bar (1e-10).
"""
import functools

import numpy as np
import pytest
import torch

from oracle import gls_oracle as O
from paper_1302_4332_amd import synth
from paper_1302_4332_amd.gls import GLSContext, GLSFunction, stream_grad_file, t2_loss
from parity_util import as_numpy, compare

pytestmark = pytest.mark.gpu
DEV = "cuda"
KEYS = ("b", "sigma2", "v", "status")


def _t(a):
    return torch.tensor(np.ascontiguousarray(a), device=DEV)


@functools.lru_cache(maxsize=2)
def _study(n, p, m):
    Phi = synth.kinship(n, n + p)
    XL = synth.covariates(n, p, n, "gauss") if p > 1 else np.empty((n, 0))
    return Phi, XL, synth.phenotype(n, n), synth.genotypes(n, 0, m, n)


def _fractional(pattern, m):
    """Which SNPs are moved off the whole numbers."""
    j = np.arange(m)
    return {"none": j < 0, "all": j >= 0, "every other": j % 2 == 1, "one": j == m - 1, "all but one": j != m // 2,
            "first 192": j < 192, "first 193": j < 193, "first 1,472": j < 1472, "first 1,473": j < 1473,
            "first 1,407": j < 1407, "first 1,408": j < 1408, "runs": (j // 200) % 2 == 0, "one in 64": j % 64 == 7, "all but one in 64": j % 64 != 7}[pattern]


def _same(a, b, what):
    for k in KEYS:
        assert np.array_equal(a[k].view(np.uint8), b[k].view(np.uint8)), f"{k}: {what}"


# n = 600, 608: 19 tiles of 32 rows, so that more than 27 of 64 SNPs are many; 608 fills the FP64 product's k stages, so
# that aligned blocks are read in place, 600 does not, so that they are copied.  m around 11 tiles of 160.
@pytest.mark.parametrize("n,p,m,pattern", [
    (608, 4, 1760, "none"), (608, 4, 1759, "all"), (608, 4, 1761, "every other"), (608, 20, 1760, "every other"),
    (600, 3, 1760, "one"), (600, 3, 1761, "all but one"), (601, 2, 1920, "runs"), (608, 1, 1800, "runs"),
    (1025, 4, 1153, "one in 64"), (1040, 4, 1153, "all but one in 64"), (2500, 4, 700, "every other"),
    # sums of 4,096 and more: lists of up to 192 columns on the kernels of few tiles, of up to 1,472 on the narrow tiles
    (4112, 3, 1600, "none"), (4112, 3, 1600, "all"), (4112, 3, 1600, "one"), (4112, 3, 1600, "all but one"),
    (4112, 3, 1600, "every other"), (4101, 3, 1600, "one in 64"), (4101, 3, 1600, "all but one in 64"),
    (4112, 3, 1600, "first 192"), (4112, 3, 1600, "first 193"), (4112, 3, 1600, "first 1,472"),
    (4101, 3, 1600, "first 1,473"), (4112, 3, 1600, "first 1,408"), (4112, 3, 1600, "first 1,407"),
])
def test_blocks_of_many_snps(n, p, m, pattern):
    Phi, XL, y, XR = _study(n, p, m)
    frac = _fractional(pattern, m)
    X = np.where(frac[:, None], XR * (1.0 / 3.0), XR)
    ctx = GLSContext(_t(Phi), 0.4, _t(XL) if p > 1 else None, _t(y), block_cols=m)
    Xd = _t(X)
    whole = as_numpy(ctx.block(Xd))
    off = torch.empty(m * n + 1, dtype=torch.float64, device=DEV)[1:].view(m, n)   # 8-byte aligned columns
    off.copy_(Xd)
    _same(as_numpy(ctx.block(off)), whole, "unaligned columns")
    for j0 in range(0, m, 97):
        j1 = min(m, j0 + 97)
        part = as_numpy(ctx.block(Xd[j0:j1]))
        _same({k: whole[k][j0:j1] for k in KEYS}, part, f"SNPs {j0}..{j1 - 1}")
    some = np.unique(np.concatenate([np.arange(8), np.arange(m - 8, m), np.arange(150, 170)]))
    if n > 4000 and pattern != "every other":
        return   # the oracle's factorization of the same study once
    compare({k: whole[k][some] for k in KEYS}, O.gls_sequence(Phi, 0.4, XL, y, X[some]), 1e-10)
    ctx.close()


@pytest.mark.parametrize("n,m", [(608, 1761), (1001, 1100)])
def test_bytes_beside_their_values(n, m):
    """Bytes above the int8 range among dosages, in a block of many SNPs."""
    Phi, XL, y, XR = _study(n, 4, m)
    G = XR.astype(np.uint8)
    G[::3, 5] = 200
    ctx = GLSContext(_t(Phi), 0.4, _t(XL), _t(y), block_cols=m)
    a, b = as_numpy(ctx.block_u8(_t(G))), as_numpy(ctx.block(_t(G.astype(np.float64))))
    _same(a, b, "bytes")
    compare({k: a[k][:40] for k in KEYS}, O.gls_sequence(Phi, 0.4, XL, y, G[:40].astype(np.float64)), 1e-10)
    ctx.close()


@pytest.mark.parametrize("m", [1727, 1728, 1729])
def test_emulation_widths(m):
    """The seven-digit product's tiles of 192 SNPs at their edge (nine tiles), against narrow blocks."""
    n = 600
    Phi, XL, y, XR = _study(n, 4, m)
    G = XR.astype(np.uint8)
    ctx = GLSContext(_t(Phi), 0.4, _t(XL), _t(y), block_cols=m, precision="int8_emu")
    Gd = _t(G)
    whole = as_numpy(ctx.block_u8(Gd))
    _same(as_numpy(ctx.block_u2(_t(synth.pack_dosages_2bit(G)))), whole, "2-bit codes")
    for j0 in range(0, m, 191):
        j1 = min(m, j0 + 191)
        _same({k: whole[k][j0:j1] for k in KEYS}, as_numpy(ctx.block_u8(Gd[j0:j1])), f"SNPs {j0}..{j1 - 1}")
    compare({k: whole[k][-40:] for k in KEYS}, O.gls_sequence(Phi, 0.4, XL, y, XR[-40:]), 1e-10)
    ctx.close()


@pytest.mark.parametrize("n", [600, 608])
def test_gradient(n):
    """The adjoint recomputes blocks of both kinds: the SNPs' gradients bitwise those of narrow blocks, whose kernels are
    those of few tiles, and the sums over SNPs equal to their rounding (1,760 terms: 1e-12)."""
    m = 1760
    Phi, XL, y, XR = _study(n, 3, m)
    X = np.where(_fractional("runs", m)[:, None], XR * (1.0 / 3.0), XR)
    grads = []
    for bc in (1760, 160):
        yt, Xt = _t(y).requires_grad_(True), _t(X).requires_grad_(True)
        h2 = torch.tensor(0.4, dtype=torch.float64, device=DEV, requires_grad=True)
        out = GLSFunction.apply(yt, Xt, h2, _t(Phi), _t(XL), bc)
        grads.append([g.cpu().numpy() for g in torch.autograd.grad(t2_loss(*out), (yt, Xt, h2))])
    (ya, xa, ha), (yb, xb, hb) = grads
    assert np.array_equal(xa.view(np.uint8), xb.view(np.uint8))
    assert np.abs(ya - yb).max() <= 1e-12 * np.abs(yb).max()
    assert abs(ha - hb) <= 1e-12 * abs(hb)


@pytest.mark.parametrize("n", [601, 608])
def test_gradient_of_bytes_in_a_file(n, tmp_path):
    """The adjoint's blocks read as bytes lie widened in a buffer of the handle, and the FP64 product reads its columns
    there: bitwise the study whose file holds the same values in FP64."""
    m = 1760
    Phi, XL, y, XR = _study(n, 3, m)
    G = XR.astype(np.uint8)
    G[::3, 5] = 200
    (tmp_path / "x.u8").write_bytes(G.tobytes())
    (tmp_path / "x.f64").write_bytes(G.astype(np.float64).tobytes())
    outs = []
    for name, fmt in (("x.u8", torch.uint8), ("x.f64", torch.float64)):
        grad = torch.empty(m, n, dtype=torch.float64).pin_memory()
        loss, yg, hg, out = stream_grad_file(_t(Phi), 0.4, _t(XL), _t(y), str(tmp_path / name), m, t2_loss,
                                             block_cols=m, fmt=fmt, XR_grad=grad)
        outs.append([np.float64(loss).reshape(1), yg.cpu().numpy(), hg.cpu().numpy().reshape(1), grad.numpy()] +
                    [t.numpy() for t in out])
    for a, b in zip(*outs):
        assert np.array_equal(np.ascontiguousarray(a).view(np.uint8), np.ascontiguousarray(b).view(np.uint8))


def test_each_product_does_its_own_columns():
    """A block of alternating whole-number and fractional SNPs takes less than the same block of fractional ones, which
    the FP64 product forms alone (about 0.65 of it; 1.3 if each product formed the other's columns as well)."""
    n, m = 5008, 4096
    Phi, XL, y, XR = _study(n, 4, m)
    ctx = GLSContext(_t(Phi), 0.4, _t(XL), _t(y), block_cols=m)
    Xf = _t(XR * (1.0 / 3.0))
    Xm = Xf.clone()
    Xm[::2] = _t(XR[::2])

    def ms(X):
        for _ in range(3):
            ctx.block(X)
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(10):
            ctx.block(X)
        b.record()
        b.synchronize()
        return a.elapsed_time(b) / 10

    f, mixed = ms(Xf), ms(Xm)
    print(f"fractional {f:.3f} ms, mixed {mixed:.3f} ms")
    ctx.close()
    assert mixed <= 0.9 * f
