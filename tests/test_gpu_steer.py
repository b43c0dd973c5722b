"""The particle step's direction for waves with a lane on flat ground, or with a gradient outside the short form's range, no
number or no direction: the plain formula's bits, and a flat lane leaves its neighbours the short form."""
import importlib.util
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.gpu
def test_direction_beside_flat_and_odd_lanes(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    spec = importlib.util.spec_from_file_location("_avl_build", os.path.join(ROOT, "paper_2506_23364_amd", "build.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    flags = [f for f in b.HIP_FLAGS if f not in ("-shared", "-fPIC", "-fvisibility=hidden")]
    exe = str(tmp_path / "steer_check")
    subprocess.run([hipcc, *flags, f"-I{ROOT}/include", os.path.join(ROOT, "tests", "support", "steer_check.hip"), "-o", exe],
                   check=True, capture_output=True, timeout=100)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=60).stdout.splitlines()
    assert len(out) == 13 * 12
    # squares in [2^-80, 2^80], and 0 (also by underflow) and NaN, whose quotients no one uses
    short = {"0x0p+0", "-0x0p+0", "0x1p-1", "0x1p-39", "0x1p+39", "0x1.b38fb8p-127", "nan"}
    for line in out:
        g, keeps, bad = line.split()
        assert bad == "0", line
        assert keeps == ("1" if g in short else "0"), line
