"""The repack and the kernels that write the prefill FFN's tables, run on the CPU.

The device sources are compiled for the host with a stand-in for the HIP runtime
(``host_kernels/hip/hip_runtime.h``: a workgroup's threads are fibers) under
AddressSanitizer, and run on buffers of exactly the sizes the workspace gives them, over
residency maps whose experts share slots too.  The driver checks the tables as the FFN
kernels read them: every group and item in its place and in range, nothing written past the
room.
"""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CLANG = "/opt/rocm/llvm/bin/clang++"


@pytest.mark.skipif(not os.path.exists(CLANG), reason="the ROCm clang++ is not here")
def test_tables_on_the_cpu(tmp_path):
    exe = tmp_path / "driver"
    src = os.path.join(HERE, "host_kernels")
    cmd = [CLANG, "-x", "c++", "-std=c++17", "-O0", "-g", "-w", "-fsanitize=address,undefined",
           "-fno-sanitize-recover=undefined", "-I", src, os.path.join(src, "driver.cpp"), "-o", str(exe)]
    built = subprocess.run(cmd, capture_output=True, text=True)
    assert built.returncode == 0, built.stderr
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0")
    env.pop("LD_PRELOAD", None)
    r = subprocess.run([str(exe)], capture_output=True, text=True, env=env, timeout=600)
    assert r.returncode == 0 and "tables ok" in r.stdout, r.stdout[-2000:] + r.stderr[-4000:]
