"""Cases that time the solver's public entry points over the sizes and forms its users run.

Sizes come from the study shapes of ``synth.WORKLOADS`` (n = 512, 4,096, 10,000 and 20,000 samples, p = 4 or 8,
blocks of 2,048 to 16,384 SNPs), from the tests (a few hundred samples, odd n and block widths, p from 1 to 20) and
from the benchmark (streams from page-locked memory, genotype bytes, the refined forms, the adjoint).

A case's ``form`` says which call it makes:

  noalloc   solve_noalloc: setup and every SNP in one call
  study     GLSContext, every SNP in blocks, close: a study from its inputs to its results
  block     one block of SNPs through a handle that is kept (GLSContext.block, .block_u8 or .block_u2 by ``data``)
  stream    the SNPs in page-locked host memory through a handle that is kept (GLSContext.stream)
  grad      GLSFunction forward and backward for the sum of squared t-statistics
  sgrad     stream_grad: the same loss with the SNPs in page-locked host memory

``data`` is how the SNPs are held: f64 (dosages 0, 1, 2), imputed (fractional expected dosages in FP64), u8
(bytes), u2 (four to a byte).
"""
import math

import torch

from paper_1302_4332_amd import gls

DEV = "cuda"
# fewest sweeps that meet the refined forms' accuracy bar
SWEEPS = {"fp64": 0, "int8_emu": 0, "fp32_ir": 1, "fp16_ir": 2, "bf16_ir": 3}


def _case(name, form, n, p, m, bc=None, data="f64", precision="fp64", h2=0.4):
    return {"name": name, "form": form, "n": n, "p": p, "m": m, "bc": bc or m, "data": data, "precision": precision,
            "h2": h2}


def listed():
    return [
        # a pilot study of a few SNPs in one call: launches and latency only
        _case("noalloc_n200", "noalloc", 200, 3, 40),
        # a small study from inputs to results
        _case("study_n512", "study", 512, 4, 2048, h2=0.5),
        # a handful of SNPs looked at again in a study of ordinary size
        _case("block_n1000_m48", "block", 1000, 4, 48),
        # odd sample count, odd block, more covariates: no dimension fits a tile
        _case("block_n2503_m1001", "block", 2503, 8, 1001),
        # imputed dosages: FP64 values that are not whole numbers
        _case("block_imputed_n5000", "block", 5000, 6, 4096, data="imputed"),
        # the main workload's block
        _case("block_n10000_m8192", "block", 10000, 4, 8192),
        # the largest sample count, eight covariates
        _case("block_n20000_m4096", "block", 20000, 8, 4096),
        # the headline use: a study's SNPs streamed from page-locked memory
        _case("stream_n10000", "stream", 10000, 4, 16384, bc=8192),
        # genotype bytes streamed through the integer form
        _case("stream_u8_int8_n10000", "stream", 10000, 4, 16384, bc=8192, data="u8", precision="int8_emu"),
        # the refined form (FP32 solves, one FP64 refinement sweep)
        _case("block_fp32_ir_n6000", "block", 6000, 4, 4096, precision="fp32_ir"),
        # differentiating a study: setup, forward, adjoint
        _case("grad_n4096", "grad", 4096, 4, 4096, h2=0.3),
        # a whole study at the main sample count, setup included
        _case("study_n10000", "study", 10000, 4, 8192),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    form = rng.choice(["noalloc", "study", "study", "block", "block", "block", "block", "stream", "stream", "grad",
                       "sgrad"])
    hi_n, hi_m = {"noalloc": (700, 256), "study": (8000, 8192), "block": (12000, 8192), "stream": (8000, 12288),
                  "grad": (4000, 4000), "sgrad": (3500, 3500)}[form]
    n = _log_int(rng, 64, hi_n)
    m = _log_int(rng, 1, hi_m)
    p = min(rng.choice([1, 2, 3, 4, 4, 4, 6, 8, 8, 12, 20]), n // 4)
    if rng.random() < 0.3:   # sizes that fill tiles
        n, m = max(64, n // 64 * 64), max(64, m // 64 * 64)
    precision = "fp64"
    data = rng.choice(["f64", "f64", "f64", "imputed"])
    if form in ("block", "stream") and rng.random() < 0.5:
        precision = rng.choice(["int8_emu", "int8_emu", "fp32_ir", "fp16_ir", "bf16_ir", "fp64"])
        data = rng.choice(["u8", "u2"]) if precision in ("int8_emu", "fp64") else data
    bc = m if form in ("block", "noalloc") else max(1, min(m, _log_int(rng, 64, 8192)))
    c = _case("", form, n, p, m, bc, data, precision, rng.choice([0.1, 0.3, 0.4, 0.5, 0.8]))
    del c["name"]
    return c


# -- inputs ----------------------------------------------------------------------------------------------------------

def _study(case, seed):
    """Phi, X_L, y and the dosages X_R (m, n) in FP64, on the GPU."""
    n, p, m = case["n"], case["p"], case["m"]
    g = torch.Generator(device=DEV).manual_seed(seed)

    def rand(*s):
        return torch.rand(*s, generator=g, device=DEV, dtype=torch.float64)

    def randn(*s):
        return torch.randn(*s, generator=g, device=DEV, dtype=torch.float64)

    def genotypes(f, rows, cols):   # Binomial(2, f)
        G = (torch.rand(rows, cols, generator=g, device=DEV) < f).double()
        G += torch.rand(rows, cols, generator=g, device=DEV) < f
        return G

    markers = 2000
    G = genotypes(0.05 + 0.45 * torch.rand(1, markers, generator=g, device=DEV), n, markers)
    G -= G.mean(0)
    G /= G.std(0, unbiased=False).clamp_min(0.05)
    Phi = (G @ G.T) / markers
    Phi = 0.5 * (Phi + Phi.T)
    Phi.diagonal().add_(1e-3)
    del G
    XL = torch.empty(n, p - 1, device=DEV, dtype=torch.float64)
    if p > 1:
        XL[:, 0] = 1.0
    if p == 4:   # intercept, sex, age
        XL[:, 1] = (rand(n) < 0.5).double()
        XL[:, 2] = 50.0 + 10.0 * randn(n)
    elif p > 2:
        XL[:, 1:] = randn(n, p - 2)
    y = randn(n)
    f = 0.05 + 0.45 * torch.rand(m, 1, generator=g, device=DEV)
    XR = genotypes(f, m, n)
    XR[:, 0] += XR.amax(1) == XR.amin(1)   # no constant column
    if case["data"] == "imputed":   # shrunk towards the mean dosage by the uncertainty of each call
        e = 0.3 * rand(m, n)
        XR = XR * (1.0 - e) + 2.0 * f.double() * e
    return Phi.contiguous(), XL, y, XR.contiguous()


def _held(case, XR):
    """The dosages as the case's user holds them."""
    if case["data"] in ("f64", "imputed"):
        return XR
    G = XR.to(torch.uint8)
    if case["data"] == "u8":
        return G
    m, n = G.shape
    q = (n + 3) // 4
    P = torch.zeros(m, 4 * q, dtype=torch.uint8, device=G.device)
    P[:, :n] = G
    P = P.view(m, q, 4)
    return (P[:, :, 0] | (P[:, :, 1] << 2) | (P[:, :, 2] << 4) | (P[:, :, 3] << 6)).contiguous()


def _outputs(m, p, **kw):
    return (torch.empty(m, p, dtype=torch.float64, **kw), torch.empty(m, dtype=torch.float64, **kw),
            torch.empty(m, dtype=torch.float64, **kw), torch.empty(m, dtype=torch.int32, **kw))


def prepare(case, seed):
    Phi, XL, y, XR = _study(case, seed)
    s = dict(case, Phi=Phi, XL=XL, y=y, X=_held(case, XR))
    opts = {"precision": case["precision"], "refine_sweeps": SWEEPS[case["precision"]]}
    if case["form"] in ("block", "stream"):
        s["ctx"] = gls.GLSContext(Phi, case["h2"], XL, y, block_cols=case["bc"], **opts)
        s["Phi"] = None
    if case["form"] in ("stream", "sgrad"):
        host = torch.empty(s["X"].shape, dtype=s["X"].dtype, pin_memory=True)
        host.copy_(s["X"])
        s["X"] = host
    if case["form"] == "stream":
        s["out"] = _outputs(case["m"], case["p"], pin_memory=True)
    if case["form"] == "noalloc":
        s["out"] = _outputs(case["m"], case["p"], device=DEV)
    if case["form"] == "grad":
        s["y"] = y.requires_grad_(True)
        s["X"] = s["X"].requires_grad_(True)
        s["h2t"] = torch.tensor(case["h2"], dtype=torch.float64, device=DEV, requires_grad=True)
    return s


def run(s):
    form = s["form"]
    if form == "noalloc":
        gls.solve_noalloc(s["Phi"], s["h2"], s["XL"], s["y"], s["X"], *s["out"], block_cols=s["bc"])
        return s["out"]
    if form == "study":
        ctx = gls.GLSContext(s["Phi"], s["h2"], s["XL"], s["y"], block_cols=s["bc"], precision=s["precision"])
        out = _outputs(s["m"], s["p"], device=DEV)
        for j in range(0, s["m"], s["bc"]):
            k = min(s["m"], j + s["bc"])
            ctx.block_into(s["X"][j:k], *(t[j:k] for t in out))
        ctx.close()
        return out
    if form == "block":
        call = {"u8": s["ctx"].block_u8, "u2": s["ctx"].block_u2}.get(s["data"], s["ctx"].block)
        return call(s["X"])
    if form == "stream":
        out, _ = s["ctx"].stream(s["X"], out=s["out"], packed=s["data"] == "u2")
        return out
    if form == "grad":
        b, s2, v = gls.GLSFunction.apply(s["y"], s["X"], s["h2t"], s["Phi"], s["XL"], s["bc"], s["precision"], 0)
        grads = torch.autograd.grad(gls.t2_loss(b, s2, v), (s["y"], s["X"], s["h2t"]))
        return (b.detach(), s2.detach(), v.detach()) + grads
    loss, yg, hg, out = gls.stream_grad(s["Phi"], s["h2"], s["XL"], s["y"], s["X"], gls.t2_loss, block_cols=s["bc"])
    return (loss, yg, hg) + tuple(out)


def work(case):
    """Each input read and each output written once; n^2 flops a SNP for a triangular product, n^3 / 3 for the
    Cholesky factor, and for a gradient two more products a SNP and the factor's adjoint."""
    n, p, m = float(case["n"]), case["p"], float(case["m"])
    elem = {"f64": 8, "imputed": 8, "u8": 1, "u2": 0.25}[case["data"]]
    nbytes = elem * n * m + m * (8 * (p + 2) + 4)
    flops = n * n * m + 2 * n * (p + 1) * m
    if case["form"] in ("block", "stream"):
        nbytes += 4 * n * n + 8 * n * p   # the factor and the whitened covariates of the handle
    else:
        nbytes += 8 * n * n + 8 * n * p
        flops += n ** 3 / 3
    if case["form"] in ("grad", "sgrad"):
        nbytes += elem * n * m * (1 if case["form"] == "grad" else 0) + 8 * n
        flops += 2 * n * n * m + n ** 3
    return {"bytes": nbytes, "flops": flops}


# -- the same values in plain torch ----------------------------------------------------------------------------------

def _forward_substitution(L, B):
    """L^-1 B by blocks of rows."""
    if L.requires_grad or B.requires_grad:
        return torch.linalg.solve_triangular(L, B, upper=False)
    out = torch.empty_like(B)
    for i in range(0, L.shape[0], 1024):
        k = min(L.shape[0], i + 1024)
        out[i:k] = torch.linalg.solve_triangular(L[i:k, i:k].contiguous(), B[i:k] - L[i:k, :i] @ out[:i], upper=False)
    return out


def _solve(Phi, h2, XL, y, XR):
    n, p = Phi.shape[0], XL.shape[1] + 1
    L = torch.linalg.cholesky(h2 * Phi + (1.0 - h2) * torch.eye(n, dtype=Phi.dtype, device=Phi.device))
    W = _forward_substitution(L, torch.cat([XL, y[:, None]], 1))
    Xt = _forward_substitution(L, XR.T)
    Wl, yt = W[:, :-1], W[:, -1]
    sbr, rb, yy = (Xt * Xt).sum(0), Xt.T @ yt, yt @ yt
    if p == 1:
        d2 = sbr
        bp = rb / d2
        b = bp[:, None]
        res = yy
    else:
        F = torch.linalg.cholesky(Wl.T @ Wl)
        z = torch.linalg.solve_triangular(F, (Wl.T @ yt)[:, None], upper=False)
        l = torch.linalg.solve_triangular(F, Wl.T @ Xt, upper=False)
        d2 = sbr - (l * l).sum(0)
        bp = (rb - (l * z).sum(0)) / d2
        bt = torch.linalg.solve_triangular(F.T, z - l * bp, upper=True)
        b = torch.cat([bt, bp[None]], 0).T
        res = yy - (z * z).sum()
    return b, (res - bp * bp * d2) / (n - p), 1.0 / d2


def exact(case, seed):
    Phi, XL, y, XR = _study(case, seed)
    if case["form"] not in ("grad", "sgrad"):
        b, s2, v = _solve(Phi, case["h2"], XL, y, XR)
        return b.contiguous(), s2, v, None
    h2 = torch.tensor(case["h2"], dtype=torch.float64, device=DEV, requires_grad=True)
    y.requires_grad_(True)
    XR.requires_grad_(True)
    b, s2, v = _solve(Phi, h2, XL, y, XR)
    loss = (b[:, -1] ** 2 / (s2 * v)).sum()
    yg, xg, hg = torch.autograd.grad(loss, (y, XR, h2))
    b, s2, v = b.detach().contiguous(), s2.detach(), v.detach()
    if case["form"] == "grad":
        return b, s2, v, yg, xg, hg
    return float(loss.detach()), yg, hg.reshape(1), b, s2, v, None
