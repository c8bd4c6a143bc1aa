"""The pool of idle streams on the CPU: failed creations, pairs that do not pass the check, the pool's bound."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_stream_pool(tmp_path):
    text = open(os.path.join(HERE, "..", "paper_1302_4332_amd", "csrc", "stream_pool.hpp")).read()
    (tmp_path / "stream_pool.hpp").write_text(text.replace("#include <hip/hip_runtime.h>", ""))
    exe = str(tmp_path / "stream_pool")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", f"-I{tmp_path}", "-o", exe,
                    os.path.join(HERE, "native", "stream_pool.cpp")], check=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout
