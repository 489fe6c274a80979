"""The exponential of the saturating cost on the host, against 80 bits (tests/host/cost_exp.cpp): its precision over all results that are
finite, and its values where they are not, at arguments of both signs (negative cost weights make them positive)."""
import math
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_exponential_of_the_saturating_cost(tmp_path):
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not found")
    from paper_2202_13638_amd import build
    exe = str(tmp_path / "cost_exp")
    r = subprocess.run(["hipcc", "--offload-arch=gfx950", "-O2", "-std=c++17", "-ffp-contract=off", "-x", "hip", "--cuda-host-only",
                        "-I", build.CSRC, os.path.join(ROOT, "tests", "host", "cost_exp.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    print(r.stdout)
    ranges = values = 0
    for line in r.stdout.splitlines():
        f = line.split()
        if f[0] == "range":
            # a correctly rounded result is off by 2^-53 = 1.1102e-16 at the most, and by 2^-53 / sqrt(3) = 6.41e-17 in the mean where all
            # results lie just past a power of two (x from 0 to 1e-3); 0.5 % more for what the last rounding is off by itself
            assert float(f[3]) <= 1.116e-16 and float(f[4]) <= 6.45e-17, line
            ranges += 1
        elif f[0] == "subnormal":
            assert float(f[1]) <= 1.0, line                    # rounded twice, by half a step each
        else:
            x, got = float(f[2]), float(f[3])
            want = math.nan if math.isnan(x) else math.inf if x > 709.7827128933841 else 0.0 if x < -745.14 else math.exp(x)
            assert got == pytest.approx(want, rel=3e-16, abs=0.0, nan_ok=True) and math.copysign(1.0, got) == 1.0 or math.isnan(x), line
            values += 1
    assert ranges == 10 and values == 20
