"""The fast transforms' lines on the CPU: the kernels' own stage code, run
item by item (tests/host/fft_driver.cpp), against the plan's dense bases for
every length and basis they are built for, both directions."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")
CSRC = os.path.join(ROOT, "paper_2406_19920_amd", "csrc")
# relative l2 error of one transform: about log2(n) <= 9 butterfly levels plus
# twiddle and normalisation, half an ulp each and adding like a random walk,
# against bases rounded to double: below 4 ulps
EPS = {8: 2.0 ** -52, 4: 2.0 ** -23}


@pytest.mark.skipif(not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"), reason="no HIP headers")
def test_lines_match_the_dense_bases(tmp_path):
    exe = tmp_path / "fft_driver"
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(HOST, "fft_driver.cpp"),
                        os.path.join(CSRC, "plan.cpp"), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout[-300:]
    rows = [line.split() for line in r.stdout.splitlines() if line.startswith("fft ")]
    assert len(rows) == 4 * (27 + 16) + 14   # refined periodic lines above 64 points in both forward arithmetics
    for _, n, basis, size, fwd, inv in rows:
        tol = 4 * EPS[int(size)]
        assert float(fwd) < tol and float(inv) < tol, (n, basis, size, fwd, inv)
