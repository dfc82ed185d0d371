"""Host checks of passes whose stages exchange register bits with lane bits
and go through per-lane LDS slots (no GPU): tests/host_checks/gate_check.cpp emulates the encoded
tables on one tile."""
import os
import subprocess

import pytest

import paper_0710_3747_amd as spq
import workloads

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def binary(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("gates") / "gate_check")
    subprocess.check_call(["g++", "-O2", "-std=c++17", os.path.join(ROOT, "tests", "host_checks", "gate_check.cpp"),
                           os.path.join(ROOT, "paper_0710_3747_amd", "csrc", "planner.cpp"), "-o", out])
    return out


CASES = [
    # name, M, couplings, prec, k, r, c, steps, observed, half tiles
    ("ladder2x9-c64-r5", 18, workloads.ladder(9), 1, 14, 5, 4, 30, 0, 1),
    ("ladder2x15-c64-r5-top-site", 30, workloads.ladder(15), 1, 14, 5, 4, 20, 29, 1),
    ("ladder2x15-c64-r6", 30, workloads.ladder(15), 1, 14, 6, 4, 20, 7, 1),
    ("ladder2x15-c64-one-gate", 30, workloads.ladder(15), 1, 14, 5, 5, 20, 0, 1),
    ("ladder2x15-c64-no-gate", 30, workloads.ladder(15), 1, 14, 5, 6, 20, 0, 1),
    ("ladder2x15-c128-k13-r4", 30, workloads.ladder(15), 2, 13, 4, 4, 20, 0, 1),
    ("ladder2x15-c128-k14", 30, workloads.ladder(15), 2, 14, 5, 4, 20, 0, 1),
    ("star17-c128-zz", 17, workloads.star(17, 3, a_over_b=0.5), 2, 13, 5, 4, 10, 5, 1),
    ("star28-blocks-c64", 28, workloads.star_m28(), 1, 14, 5, 4, 2, 0, 1),
    ("two-site-bond-c64", 15, [(3, 11, 0.0, 1.0)], 1, 14, 5, 4, 3, 14, 1),
    ("ladder2x9-c64-k10", 18, workloads.ladder(9), 1, 10, 2, 4, 30, 0, 0),
    ("star15-c64-k11-zz", 15, workloads.star(15, 3, a_over_b=-2.0), 1, 11, 3, 4, 10, 7, 0),
    ("ladder2x9-c64-k12", 18, workloads.ladder(9), 1, 12, 4, 4, 30, 17, 0),
    ("chain14-c128-k12-c2", 14, workloads.chain(14), 2, 12, 4, 2, 30, 0, 0),
    # passes of one stage that exchanges
    ("chain18-c64-half-c2", 18, workloads.chain(8), 1, 14, 5, 2, 3, 0, 1),
    ("star17-c128-k12", 17, workloads.star(17, 3), 2, 12, 4, 4, 10, 0, 0),
    # one-workgroup plans (k bits, sites past M are padding)
    ("resident-ladder2x5", 10, workloads.ladder(5), 1, 10, 4, 0, 5, 0, 2),
    ("resident-ladder2x5-no-steps", 10, workloads.ladder(5), 1, 10, 4, 0, 0, 3, 2),
    ("resident-bond", 2, workloads.single_bond(0, 1), 2, 10, 4, 0, 4, 1, 2),
    ("resident-one-site", 1, [], 1, 10, 4, 0, 3, 0, 2),
    ("resident-chain11-c128", 11, workloads.chain(11), 2, 11, 4, 0, 1, 5, 2),
    ("resident-dipolar13", 13, workloads.star(13, 7, a_over_b=-2.0), 1, 13, 4, 0, 3, 12, 2),
    ("resident-star14", 14, workloads.star(14, 7), 1, 14, 4, 0, 2, 0, 2),
    ("resident-star13-r5", 13, workloads.star(13, 7), 1, 13, 5, 0, 2, 0, 2),
    ("resident-duplicates", 6, workloads.chain(6) + [(0, 1, 0.0, 1.0), (1, 0, 0.0, 0.5)], 2, 10, 4, 0, 4, 1, 2),
    ("chain13-c64-one-wave", 13, workloads.chain(13), 1, 11, 5, 4, 30, 0, 0),
    # 512 lanes of 16 amplitudes, the default at M = 21
    ("star21-c64-k13", 21, workloads.star(21, 3), 1, 13, 4, 4, 3, 20, 0),
    ("ladder2x10-dangling-c64-k13-zz", 21, workloads.ladder(10, a_over_b=0.5) + [(0, 20, 0.0, 0.3)], 1, 13, 4, 4, 30, 0, 0),
    ("chain22-c64-r5", 22, workloads.chain(22), 1, 14, 5, 4, 30, 11, 1),
    ("star23-c64-r5", 23, workloads.star(23, 3), 1, 14, 5, 4, 3, 0, 1),
    ("chain21-c128-k13", 21, workloads.chain(21, a_over_b=-2.0), 2, 13, 5, 4, 30, 0, 1),
    # what half tiles of every shape exchange through in a run (test_host_plan
    # checks the one layout that they could share)
    ("ladder2x15-c64-k14r5c4-1000", 30, workloads.ladder(15), 1, 14, 5, 4, 1000, 0, 1),
    ("ladder2x15-c64-k14r5c5-3steps", 30, workloads.ladder(15), 1, 14, 5, 5, 3, 0, 1),
    ("ladder2x15-c64-k14r6c4-100", 30, workloads.ladder(15), 1, 14, 6, 4, 100, 0, 1),
    ("ladder2x15-c128-k13r4c4-100", 30, workloads.ladder(15), 2, 13, 4, 4, 100, 0, 1),
    ("ladder2x15-c128-k13r5c4-100", 30, workloads.ladder(15), 2, 13, 5, 4, 100, 0, 1),
    ("ladder2x15-c128-k14r5c4-100", 30, workloads.ladder(15), 2, 14, 5, 4, 100, 0, 1),
    ("star28-c64-k14r5c6", 28, workloads.star(28, 33), 1, 14, 5, 6, 12, 0, 1),
    ("star28-blocks-c64-k14r6c4", 28, workloads.star_m28(), 1, 14, 6, 4, 12, 0, 1),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_register_lane_exchanges(case, binary):
    _, M, J, prec, k, r, c, steps, obs, half = case
    inp = f"{M} {prec} {k} {r} {c} {steps} {obs} {half}\n" + "".join(f"{i} {j} {a!r} {b!r}\n" for i, j, a, b in J)
    p = subprocess.run([binary], input=inp, capture_output=True, text=True, timeout=300)
    assert p.returncode == 0 and " failures 0" in p.stdout, p.stdout


@pytest.mark.parametrize("M,steps,tile", [(26, 20, 13), (28, 2, 13), (28, 21, 14), (30, 10, 14)])
def test_double_precision_tiles_follow_the_launches_they_save(M, steps, tile):
    args = (spq.SPIN_C128, M, workloads.ladder(M // 2), 0.05, steps, 0)
    got = spq.spin_describe_plan(*args, spq.Options())
    n = {k: spq.spin_describe_plan(*args, spq.Options(tile_bits=k))["launches"] for k in (13, 14)}
    assert got["tile_bits"] == tile and got["launches"] == n[tile]
    assert (10 * n[13] > 13 * n[14]) == (tile == 14) or M < 27


def test_batch_kernel_buffer_holds_what_its_problems_touch(tmp_path):
    """One-workgroup problems of the batch kernel exchange in padded rows; the
    kernel's LDS buffer holds them for both precisions and tile modes."""
    out = str(tmp_path / "batch_lds_check")
    subprocess.check_call(["g++", "-O2", "-std=c++17", os.path.join(ROOT, "tests", "host_checks", "batch_lds_check.cpp"),
                           "-o", out])
    p = subprocess.run([out], capture_output=True, text=True, timeout=60)
    assert p.returncode == 0, p.stdout


def test_gang_meetings_across_the_wrap_of_their_counter(tmp_path):
    """A gang's counter of arrivals wraps in a long run: no meeting is passed
    early and none waits for ever; a wait ends by time only when nothing moves."""
    out = str(tmp_path / "gang_check")
    subprocess.check_call(["g++", "-O2", "-std=c++17", os.path.join(ROOT, "tests", "host_checks", "gang_check.cpp"),
                           "-o", out])
    p = subprocess.run([out], capture_output=True, text=True, timeout=60)
    assert p.returncode == 0, p.stdout


def test_calls_kept_are_bounded(tmp_path):
    """What is kept of past batched calls is bounded in number and bytes."""
    out = str(tmp_path / "kept_check")
    subprocess.check_call(["g++", "-O2", "-std=c++17", os.path.join(ROOT, "tests", "host_checks", "kept_check.cpp"),
                           "-o", out])
    p = subprocess.run([out], capture_output=True, text=True, timeout=60)
    assert p.returncode == 0, p.stdout
