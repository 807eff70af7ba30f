"""The pseudo-potential of FP32 population storage, psi(rho_ref + d) - psi(rho_ref)
= -E expm1(-d / rho_0): the kernels' function compiled for the host is within the
1 ulp to which the mathematical library gives expm1f, and keeps its limits at
infinite arguments (E from above, minus infinity from below)."""
import os
import re
import subprocess

from paper_1004_5058_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_fp32_psi_is_as_exact_as_expm1(tmp_path):
    exe = str(tmp_path / "psi_bound")
    cmd = [build.HIPCC, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-ffp-contract=on", "-I" + build.CSRC,
           "-I" + os.path.join(build.ROOT, "include"), os.path.join(HERE, "psi", "psi_bound.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    print(r.stdout)
    assert float(re.search(r"worst ([0-9.naif]+) ulp", r.stdout).group(1)) <= 1.0
    assert "+inf 1, -inf -inf" in r.stdout
