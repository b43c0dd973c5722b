"""What the autotuner keeps one choice for: calls that run different kernels never share one, calls of one size class do."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def keys(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("keys") / "tuning_keys")
    cxx = shutil.which("g++") or shutil.which("c++")
    subprocess.run([cxx, "-std=c++17", "-Wall", os.path.join(HERE, "support", "tuning_keys.cpp"), "-o", exe], check=True,
                   capture_output=True, timeout=120)

    def run(*problems):
        args = [str(a) for p in problems for a in p]
        return subprocess.run([exe, *args], check=True, capture_output=True, text=True, timeout=20).stdout.splitlines()
    return run


@pytest.mark.parametrize("n,cap,P,S", [(1, 0, 1, 0), (45492, 600, 10, 1000), (1 << 20, 5000, 128, 3000)])
def test_velocity_forward_has_a_choice_of_its_own(keys, n, cap, P, S):
    dep, vel, back, again = keys(("s", 2, n, cap, P, S, 0), ("s", 2, n, cap, P, S, 1), ("s", 3, n, cap, P, S, 0),
                                 ("s", 2, n, cap, P, S, 1))
    assert len({dep, vel, back}) == 3 and vel == again
    assert dep.split()[1] == vel.split()[1] == "2" and back.split()[1] == "3"  # the kind, which the overrides read


def test_sizes_share_a_choice_by_powers_of_two(keys):
    a, b, c = keys(("s", 2, 40000, 600, 10, 1000, 1), ("s", 2, 65535, 1000, 15, 1022, 1), ("s", 2, 65536, 600, 10, 1000, 1))
    assert a == b != c
    a, b, c = keys(("t", 0, 40000, 1, 10, 1000, 0), ("t", 0, 65535, 1, 15, 1022, 0),
                   ("t", 1, 40000, 1, 10, 1000, 0))
    assert a == b != c


def test_runout_stop_has_a_choice_of_its_own(keys):
    off, on, batch_off, batch_on = keys(*[("t", b, 1 << 22, 4, 32, 2000, r) for b in (0, 1) for r in (0, 1)])
    assert off != on
    assert batch_off == batch_on != off  # a batch always has the stop compiled in
