"""Batched launches that need no gang: they run beside other work of the device,
small ones can be captured, and problems without couplings share the slots."""
import time

import pytest

import workloads
import paper_0710_3747_amd as spq
from gpu_helpers import TOL_P, note, torch_dtype

pytestmark = pytest.mark.gpu
C64, C128 = spq.SPIN_C64, spq.SPIN_C128


def problems(prec, sizes, steps, couplings=None, first=1):
    import torch
    out = []
    for q, M in enumerate(sizes):
        out.append({"psi": torch.zeros(2 ** max(M, 1), dtype=torch_dtype(prec), device="cuda"), "M": M,
                    "couplings": workloads.star(M, 3 + q % 3) if couplings is None else couplings,
                    "observed_site": M - 1, "polarized_site": 0, "seed": first + q,
                    "P": torch.zeros(steps + 1, dtype=torch.float64, device="cuda"),
                    "N": torch.zeros(steps + 1, dtype=torch.float64, device="cuda")})
    return out


def check_against_single_runs(prec, ps, dt, steps):
    import torch
    for p in ps:
        psi, P, N = torch.empty_like(p["psi"]), torch.zeros_like(p["P"]), torch.zeros_like(p["N"])
        spq.spin_init_random_phase(psi, p["M"], p["polarized_site"], p["seed"])
        spq.spin_trotter_evolve_ex(psi, p["M"], p["couplings"], dt, steps, p["observed_site"], P, N)
        torch.cuda.synchronize()
        assert float((P - p["P"]).abs().max()) < TOL_P[prec] and float((N - p["N"]).abs().max()) < TOL_P[prec]
        assert float((psi - p["psi"]).abs().max()) < TOL_P[prec]


@pytest.mark.parametrize("prec", [C64, C128])
def test_batches_of_every_small_size_match_single_runs(prec):
    """1 to 13 sites in one call: the waves of their own and the persistent launch."""
    note("small sizes", prec)
    dt, steps = 0.05, 6
    ps = problems(prec, list(range(1, 14)) + [4, 2, 1, 5], steps)
    spq.spin_trotter_evolve_batch(ps, prec, dt, steps)
    check_against_single_runs(prec, ps, dt, steps)


@pytest.mark.parametrize("prec", [C64, C128])
def test_small_problems_can_be_captured_once_their_tables_are_there(prec):
    """Replayed three times with eager calls between."""
    import torch
    note("captured batch", prec)
    dt, steps = 0.05, 7
    ps = problems(prec, [4, 3, 2, 1, 4, 4], steps)
    side = torch.cuda.Stream()
    spq.spin_trotter_evolve_batch(ps, prec, dt, steps, stream=side.cuda_stream)
    torch.cuda.synchronize()
    want = [(p["psi"].clone(), p["P"].clone(), p["N"].clone()) for p in ps]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        spq.spin_trotter_evolve_batch(ps, prec, dt, steps, stream=side.cuda_stream)
    other = problems(prec, [4, 8, 15], steps, first=9)
    for _ in range(3):
        for p in ps:
            p["psi"].zero_(), p["P"].zero_(), p["N"].zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for p, (psi, P, N) in zip(ps, want):
            assert torch.equal(p["psi"], psi) and torch.equal(p["P"], P) and torch.equal(p["N"], N)
        spq.spin_trotter_evolve_batch(other, prec, dt, steps)
    torch.cuda.synchronize()
    assert spq.spin_batch_status() == 0


@pytest.mark.parametrize("M", [4, 10])
def test_batches_without_gangs_overlap(M):
    """A short call on one stream ends while a long one on another still runs."""
    import torch
    note("overlap", M)
    long_steps = 400000 if M == 4 else 100000       # a third of a second and more
    long, short = problems(C64, [M], long_steps), problems(C64, [M], 3)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    # tables first, with the long one's number of steps
    spq.spin_trotter_evolve_batch(short, C64, 0.01, 3, stream=b.cuda_stream)
    spq.spin_trotter_evolve_batch(long, C64, 0.01, long_steps, stream=a.cuda_stream)
    torch.cuda.synchronize()
    spq.spin_trotter_evolve_batch(long, C64, 0.01, long_steps, stream=a.cuda_stream)
    spq.spin_trotter_evolve_batch(short, C64, 0.01, 3, stream=b.cuda_stream)
    b.synchronize()
    running = not a.query()
    torch.cuda.synchronize()
    assert running


@pytest.mark.parametrize("gangs_first", [False, True])
def test_gangs_run_beside_no_other_batch(gangs_first):
    """A gang's launch needs all its slots: it starts after a call without gangs
    that another stream runs, and such a call starts after it."""
    import torch
    note("gangs and others", gangs_first)
    dt = 0.01
    M, long_steps = (15, 10000) if gangs_first else (10, 100000)      # about a third of a second
    J = workloads.chain(M)
    long, short = problems(C64, [M], long_steps, J), problems(C64, [10 if gangs_first else 15], 3)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    spq.spin_trotter_evolve_batch(short, C64, dt, 3, stream=b.cuda_stream)
    spq.spin_trotter_evolve_batch(long, C64, dt, long_steps, stream=a.cuda_stream)
    torch.cuda.synchronize()
    spq.spin_trotter_evolve_batch(long, C64, dt, long_steps, stream=a.cuda_stream)
    assert not a.query()
    spq.spin_trotter_evolve_batch(short, C64, dt, 3, stream=b.cuda_stream)
    b.synchronize()
    assert a.query()
    assert spq.spin_batch_status() == 0
    check_against_single_runs(C64, short, dt, 3)


def test_problems_without_couplings_share_the_slots():
    """512 problems of 11 sites without couplings take less time than with a chain."""
    import torch
    note("uncoupled")
    steps, n, M = 50, 512, 11
    took = []
    for J in ([], workloads.chain(M)):
        ps = problems(C64, [M] * n, steps, couplings=J)
        best = 1e9
        for _ in range(3):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            spq.spin_trotter_evolve_batch(ps, C64, 0.05, steps)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
        took.append(best)
    assert took[0] <= took[1], took


def test_calls_with_new_seeds_do_not_pile_up():
    """More calls with new seeds than are kept, on two streams: the states stay
    right and the device's free memory stops falling."""
    import torch
    note("new seeds")
    dt, steps, M = 0.05, 2, 14
    ps = problems(C64, [M], steps, couplings=workloads.chain(M))
    streams = [torch.cuda.Stream() for _ in range(2)]
    spq.spin_release_caches()
    free = []
    for turn in range(3):
        for q in range(1100):
            ps[0]["seed"] = 1100 * turn + q
            spq.spin_trotter_evolve_batch(ps, C64, dt, steps, stream=streams[q % 2].cuda_stream)
            if q % 100 == 99:
                torch.cuda.synchronize()
        check_against_single_runs(C64, ps, dt, steps)
        free.append(torch.cuda.mem_get_info()[0])
    assert free[2] == free[1]
    assert spq.spin_batch_status() == 0
