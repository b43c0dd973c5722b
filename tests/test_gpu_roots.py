"""The particle step's short square roots and quotients by a root equal the compiler's correctly rounded ones for every
binary32 argument of their range (exhaustive, on the GPU: they start from the hardware's estimate)."""
import importlib.util
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.gpu
def test_short_roots_are_correctly_rounded(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    spec = importlib.util.spec_from_file_location("_avl_build", os.path.join(ROOT, "paper_2506_23364_amd", "build.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    flags = [f for f in b.HIP_FLAGS if f not in ("-shared", "-fPIC", "-fvisibility=hidden")]
    exe = str(tmp_path / "root_check")
    subprocess.run([hipcc, *flags, f"-I{ROOT}/include", os.path.join(ROOT, "tests", "support", "root_check.hip"), "-o", exe],
                   check=True, capture_output=True, timeout=100)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=60).stdout.splitlines()
    assert len(out) == 11
    for line in out:
        assert line.split()[3:] == ["0", "0", "0"], line
