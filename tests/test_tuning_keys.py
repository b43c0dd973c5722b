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


@pytest.mark.parametrize("P", [1, 2, 4, 7, 8, 9, 10, 32, 100, 1 << 20, (1 << 32) - 1])
def test_velocity_rule_by_size(keys, P):
    # straight for sure, straight first if chosen, through the table for sure: in this order with growing size, at every P
    sizes = sorted({1, 3071, 3072, 3073, (1 << 32) - 1, *(max(1, c * 3072 // P ** 2 + d) for c in (128, 1024) for d in (-1, 0, 1))})
    got = [int(x) for x in keys(*[("v", s, P, 0, 0, 0, 0) for s in sizes])]
    for s, g in zip(sizes, got):
        few = s * P * P <= 128 * 3072 if P <= 8 else False
        assert g == (2 if s <= 3072 or few else 1 if P <= 8 and s * P * P <= 1024 * 3072 else 0), (s, P)
    assert got == sorted(got, reverse=True)


def test_velocity_rule_at_the_measured_sizes(keys):
    # where straight was faster on short paths and the table on long ones the tuner decides
    sizes = ((2470, 10, 2), (1600, 8, 2), (80000, 1, 2), (40000, 4, 1), (80000, 4, 1), (40000, 8, 1), (10000, 8, 1),
             (160000, 4, 1), (320000, 4, 0), (12000, 40, 0), (6000, 10, 0))
    got = [int(x) for x in keys(*[("v", s, P, 0, 0, 0, 0) for s, P, _ in sizes])]
    assert got == [w for _, _, w in sizes]
