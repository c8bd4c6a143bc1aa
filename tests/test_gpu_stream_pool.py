"""Stream pairs pass from closed handles to new ones: more handles than the pool keeps, open together and in threads."""
import threading

import numpy as np
import pytest
import torch

from paper_1302_4332_amd import synth
from paper_1302_4332_amd.gls import GLSContext

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("threads,rounds", [(1, 7), (6, 3)])
def test_streams_of_handles_opened_and_closed(threads, rounds):
    m = 300
    st = synth.make_study("c0_small", m=m)
    Phi, XL, y = (torch.tensor(np.ascontiguousarray(a), device=DEV) for a in (st.Phi, st.XL, st.y))
    host = torch.from_numpy(st.snps(0, m)).pin_memory()
    torch.cuda.synchronize()

    def study():
        ctx = GLSContext(Phi, st.w.h2, XL, y, block_cols=100)
        out = [t.numpy().copy() for t in ctx.stream(host)[0]]
        ctx.close()
        return out

    ref, got = study(), []

    def work():
        for _ in range(rounds):
            got.append(study())

    ts = [threading.Thread(target=work) for _ in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join(60)
    assert len(got) == threads * rounds
    for out in got:
        for a, b in zip(out, ref):
            assert np.array_equal(a.view(np.uint8), b.view(np.uint8))
