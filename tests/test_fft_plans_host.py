"""The cheapest FFT plans (composite radices among them) on the CPU, for every
length the passes take: the transform of the plans with the simple radices."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("flags", [["-O2"], ["-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all"]])
def test_cheapest_plans(flags, tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "fft_plan_driver")
    r = subprocess.run([gxx, "-std=c++17", "-w", *flags, "-I", os.path.join(ROOT, "paper_1203_4874_amd", "csrc"),
                        os.path.join(ROOT, "tests", "host", "fft_plan_driver.cpp"), "-o", exe], capture_output=True, text=True)
    if r.returncode != 0 and len(flags) > 1:
        pytest.skip("sanitizer runtime not available: " + r.stderr[-200:])
    assert r.returncode == 0, r.stderr
    lines = subprocess.run([exe], capture_output=True, text=True, check=True).stdout.split("\n")[:-1]
    assert len(lines) == 2048
    smooth = 0
    for line in lines:
        n, passes, *err = line.split()
        if passes == "-1":
            continue
        smooth += 1
        # both within the simple radices' bound of a library transform (1e-14)
        assert float(err[0]) <= 2e-14, line
        assert int(passes) <= 4, line
    assert smooth == sum(2 ** a * 3 ** b * 5 ** c * 7 ** d <= 2048 for a in range(12) for b in range(7)
                         for c in range(5) for d in range(4))
