"""Host check of the single-precision rotation coefficients (no GPU):
tests/host_checks/rounding_check.cpp adds up, per pair of sites, by how much
the rotations of a plan are off orthogonal and off their angle."""
import os
import subprocess

import pytest

import workloads

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def binary(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("rounding") / "rounding_check")
    subprocess.check_call(["g++", "-O2", "-std=c++17", os.path.join(ROOT, "tests", "host_checks", "rounding_check.cpp"),
                           os.path.join(ROOT, "paper_0710_3747_amd", "csrc", "planner.cpp"), "-o", out])
    return out


@pytest.mark.parametrize("name,M,J,k,r,half,steps", [
    ("ladder2x9-small-tiles", 18, workloads.ladder(9), 12, 4, 0, 40),
    ("ladder2x12", 24, workloads.ladder(12), 14, 6, 1, 60),
    ("ladder2x15", 30, workloads.ladder(15), 14, 6, 1, 20),
    ("ladder2x15-long", 30, workloads.ladder(15), 14, 6, 1, 120),
    ("star16", 16, workloads.star(16, 3), 11, 3, 0, 30),
    ("strong-bonds", 16, [(i, i + 1, 0.0, 90.0 + i) for i in range(15)], 11, 3, 0, 30),
    ("weak-bonds", 16, [(i, i + 1, 0.0, 1e-6 * (i + 1)) for i in range(15)] + [(0, 15, 0.0, 0.0)], 11, 3, 0, 30),
])
def test_rounding_of_a_pair_does_not_add_up(binary, name, M, J, k, r, half, steps):
    inp = f"{M} {k} {r} {half} {steps}\n" + "".join(f"{i} {j} {b!r}\n" for i, j, _, b in J)
    p = subprocess.run([binary], input=inp, capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stdout
