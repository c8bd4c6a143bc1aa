"""Streams whose blocks are copied and solved in parts, and that copies and solves overlap for every kind of SNP.

Blocks of whole-number SNPs in a GLS_FP64 handle are copied in up to four parts of
64 MB or more; blocks that look otherwise are copied whole.  The outputs are
those of GLSContext.block whatever the parts.  Overlap is measured against what
the stream would take without it: the copies and the solves one after another.
"""
import numpy as np
import pytest
import torch

from paper_1302_4332_amd import synth
from paper_1302_4332_amd.gls import GLSContext

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _t(a):
    return torch.tensor(np.ascontiguousarray(a), device=DEV)


@pytest.mark.parametrize("kind", ["whole", "a few fractional", "every other"])
@pytest.mark.parametrize("n,bc,m,col0", [(2050, 16384, 20001, 0), (4100, 4100, 12345, 777)])
def test_parts_equal_blocks(n, bc, m, col0, kind):
    """Two to four parts, ragged last blocks, a resumed stream: bitwise the block call.  "A few fractional" SNPs differ from
    whole numbers at single samples that the stream's look at the block need not meet."""
    Phi, XL, y = synth.kinship(n, n), synth.covariates(n, 4, n, "gauss"), synth.phenotype(n, n)
    X = torch.from_numpy(synth.genotypes(n, 0, m, n)).pin_memory()
    if kind == "a few fractional":
        X[5::331, n // 2 + 1] += 0.25
    elif kind == "every other":
        X[::2] *= 1.0 / 3.0
    ctx = GLSContext(_t(Phi), 0.4, _t(XL), _t(y), block_cols=bc)
    (b, s2, v, st), stats = ctx.stream(X, col0=col0)
    assert stats.blocks > 1
    for j0 in range(col0, m, 3000):
        j1 = min(m, j0 + 3000)
        ref = ctx.block(X[j0:j1].to(DEV))
        for got, want in zip((b, s2, v, st), ref):
            assert np.array_equal(got[j0:j1].numpy().view(np.uint8), want.cpu().numpy().view(np.uint8)), (j0, j1)
    ctx.close()


@pytest.mark.parametrize("kind", ["whole", "fractional"])
def test_copies_and_solves_overlap(kind):
    """Against a serial stream of the same study, which takes its copies and then its solves: the overlapped one is
    shorter by at least half of the shorter of the two (all of it, less the opening copy and the last solve, if nothing
    holds either up).  With fractional SNPs a block's copy takes about as long as its solve."""
    m = 16384
    st = synth.make_study("c1_n10k_m100k", m=m)
    Phi, XL, y = (_t(a) for a in (st.Phi, st.XL, st.y))
    host = torch.from_numpy(st.snps(0, m)).pin_memory()
    if kind == "fractional":
        host *= 1.0 / 3.0
    kw = dict(block_cols=8192)
    serial = GLSContext(Phi, st.w.h2, XL, y, serial_stream=True, **kw)
    ref, s = min((serial.stream(host) for _ in range(3)), key=lambda r: r[1].wall_ms)
    serial.close()
    copies = s.wall_ms - s.compute_ms   # a serial stream's compute_ms is its solves alone
    ctx = GLSContext(Phi, st.w.h2, XL, y, **kw)
    for k in range(4):
        out, stats = ctx.stream(host)
        print(f"{kind} pass {k}: wall {stats.wall_ms:.1f} ms; serial {s.wall_ms:.1f}, solves {s.compute_ms:.1f}",
              flush=True)
        assert stats.wall_ms <= s.wall_ms - 0.5 * min(copies, s.compute_ms)
        for a, b in zip(out, ref):
            assert np.array_equal(a.numpy().view(np.uint8), b.numpy().view(np.uint8))
    ctx.close()
