"""The factorization's diagonal block on the CPU: its result must not depend on which wave runs ahead.

The kernel's own source runs with its waves in several orders (native/leaf_waves.cpp).  Each order has to give the
same bits, and the factor and its inverse have to match numpy's.
"""
import os
import re
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_1302_4332_amd", "csrc")


@pytest.fixture(scope="module")
def emulator(tmp_path_factory):
    d = tmp_path_factory.mktemp("leaf")
    text = open(os.path.join(CSRC, "setup_kernels.hpp")).read()
    text = re.sub(r"asm volatile\([^;]*\);", "", text).replace("#include <hip/hip_runtime.h>", "")
    (d / "setup_kernels.hpp").write_text(text)
    exe = d / "leaf_waves"
    subprocess.run(["g++", "-O1", "-std=c++17", "-w", f"-I{d}", "-o", str(exe), os.path.join(HERE, "native", "leaf_waves.cpp")],
                   check=True, timeout=300)
    return str(exe)


def test_any_wave_may_run_ahead(emulator):
    rng = np.random.default_rng(7)
    G = rng.standard_normal((128, 160))
    M = G @ G.T / 160 + 0.5 * np.eye(128)
    L = np.linalg.cholesky(M)
    ref = None
    for order in ("76543210", "01234567", "10234567", "20134567", "31720645"):
        r = subprocess.run([emulator, order], input=M.tobytes(order="F"), capture_output=True, timeout=120)
        assert r.returncode == 0, order
        out = np.frombuffer(r.stdout).reshape(2, 128, 128).transpose(0, 2, 1)
        if ref is None:
            ref = r.stdout
            # the largest entry of the error of either factor: 128 sums of 128 products, condition below 100
            assert np.abs(out[0] - L).max() <= 1e-13
            assert np.abs(np.tril(out[1]) @ L - np.eye(128)).max() <= 1e-12
        assert r.stdout == ref, f"waves in the order {order}"
