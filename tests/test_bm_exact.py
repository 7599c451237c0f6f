"""Host check that both Box-Muller generators of the FP64 normals (rows of a
table; polynomials alone, in the LB pass) are no less exact than a series over
the whole octave and octant with an IEEE division and ln 2 in two parts, whose
errors against extended precision are, in units of 2^-52: logarithm 0.266 rms and
1.023 at worst, sine and cosine 0.157 and 0.760, a normal 0.392 rms."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
RMS = {"log": 0.266, "sin": 0.157, "cos": 0.157, "z": 0.392}
WORST = {"log": 1.023, "sin": 0.760, "cos": 0.760, "edge": 1.023}


@pytest.mark.parametrize("opt", ["-O0", "-O2"])
def test_generators_are_as_exact_as_the_series(tmp_path, opt):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "bm_exact_check")
    res = subprocess.run([hipcc, opt, "-std=c++17", "-I",
                          os.path.join(ROOT, "paper_1104_0078_amd", "csrc"),
                          os.path.join(ROOT, "tests", "bm_exact_check.cpp"), "-o", exe],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    out = subprocess.run([exe, "1000000"], capture_output=True, text=True, check=True).stdout
    vals = {l.split()[0]: float(l.split()[1]) for l in out.strip().splitlines()}
    print(vals)
    for gen in ("rows", "poly"):
        for what, bar in RMS.items():
            assert vals["%s_%s_rms" % (gen, what)] <= bar, (gen, what)
        for what, bar in WORST.items():
            assert vals["%s_%s_max" % (gen, what)] <= bar, (gen, what)
