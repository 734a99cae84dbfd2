"""The repack and the kernels that write the prefill FFN's tables, run on the CPU.

The device sources are compiled for the host with a stand-in for the HIP runtime
(``host_kernels/hip/hip_runtime.h``: a workgroup's threads are fibers) under
AddressSanitizer, and run on buffers of exactly the sizes the workspace gives them, over
residency maps whose experts share slots too.  The driver checks the tables as the FFN
kernels read them: every group and item in its place and in range, nothing written past the
room.  A second program records which kernels the router's launch code picks, and the GPU
tests' shapes have to reach each of them.
"""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CLANG = "/opt/rocm/llvm/bin/clang++"


def build(tmp_path, name):
    exe = tmp_path / name
    src = os.path.join(HERE, "host_kernels")
    cmd = [CLANG, "-x", "c++", "-std=c++17", "-O0", "-g", "-w", "-fsanitize=address,undefined",
           "-fno-sanitize-recover=undefined", "-I", src, os.path.join(src, name + ".cpp"), "-o", str(exe)]
    built = subprocess.run(cmd, capture_output=True, text=True)
    assert built.returncode == 0, built.stderr
    return exe


def run(exe, text=None):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0")
    env.pop("LD_PRELOAD", None)
    r = subprocess.run([str(exe)], input=text, capture_output=True, text=True, env=env, timeout=600)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    return r.stdout


@pytest.mark.skipif(not os.path.exists(CLANG), reason="the ROCm clang++ is not here")
def test_tables_on_the_cpu(tmp_path):
    assert "tables ok" in run(build(tmp_path, "driver"))


@pytest.mark.skipif(not os.path.exists(CLANG), reason="the ROCm clang++ is not here")
def test_route_cases_reach_every_kernel(tmp_path):
    from test_gpu_route_tiles import CASES
    out = run(build(tmp_path, "route_driver"), "".join(" ".join(map(str, c)) + "\n" for c in CASES)).splitlines()
    assert len(out) == len(CASES) + 1
    picked = {w for line in out[:-1] for w in line.split()}
    print(sorted(picked))
    assert {w.rsplit(":", 1)[0] for w in picked} == set(out[-1].split()[1:])
    rows = {(w.split(":")[0], int(w.split(":")[2])) for w in picked if w.split(":")[1].endswith("true")}
    assert rows == {(dt, r) for dt in ("bf16", "f32") for r in (8, 16, 32)}
