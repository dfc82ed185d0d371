"""The states around the limits of one workgroup and of the small tiles: the
default choice against the oracle's Trotter loop, and the one-launch plan that
calls under stream capture and allocation-free calls take instead."""
import ctypes

import numpy as np
import pytest

import oracle
import workloads
from oracle import cref
import paper_0710_3747_amd as spq
from gpu_helpers import TOL_P, assert_state_close, gpu_evolve, gpu_profile, note, torch_dtype
from test_zz_no_alloc import _run

pytestmark = pytest.mark.gpu
C64, C128 = spq.SPIN_C64, spq.SPIN_C128


@pytest.mark.parametrize("prec", [C128, C64])
@pytest.mark.parametrize("phases", [False, True])
@pytest.mark.parametrize("M", [11, 12, 13, 14, 15, 16, 17, 18, 19])
def test_default_shapes_match_the_oracle(prec, phases, M):
    note("dispatch", M, prec, phases)
    J = workloads.star(M, 7, a_over_b=-2.0 if phases else 0.0)
    dt, steps = 0.03, 3
    ref = np.ascontiguousarray(oracle.random_phase_state(M, M - 1, 5))
    P0, N0 = cref.trotter_run(ref, M, J, dt, steps, M - 1)
    P, N, psi, _ = gpu_evolve(prec, M, J, dt, steps, M - 1, polarized=M - 1, seed=5)
    assert np.abs(P - P0).max() < TOL_P[prec]
    assert np.abs(N / N0 - 1).max() < TOL_P[prec]
    assert_state_close(psi, ref, prec)


@pytest.mark.parametrize("prec,M", [(C64, 12), (C64, 14), (C128, 13)])
def test_one_launch_plan_serves_captured_and_allocation_free_calls(prec, M):
    """Prepared with one number of steps, called with another; replayed three
    times with eager calls between."""
    import torch
    note("one launch", M, prec)
    lib = spq.load_library()
    J = workloads.star(M, 7, a_over_b=-2.0)
    dt, steps = 0.03, 4
    spq.spin_prepare_plan(prec, M, J, dt, steps + 3, 0, None)
    psi = torch.empty(2 ** M, dtype=torch_dtype(prec), device="cuda")
    P = torch.zeros(steps + 1, dtype=torch.float64, device="cuda")
    N = torch.zeros_like(P)
    spq.spin_init_random_phase(psi, M, 0, 2)
    start = psi.clone()
    assert _run(lib, "spin_trotter_evolve_noalloc", psi, prec, M, J, dt, steps, 0, P, N, None, torch) == 0
    torch.cuda.synchronize()
    want, wantP = psi.clone(), P.clone()
    want_np = want.cpu().numpy().astype(np.complex128)
    Pe, _, psie, _ = gpu_evolve(prec, M, J, dt, steps, 0, polarized=0, seed=2)
    assert np.abs(Pe - wantP.cpu().numpy()).max() < TOL_P[prec]
    assert_state_close(psie, want_np, prec)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        spq.spin_trotter_evolve_ex(psi, M, J, dt, steps, 0, P, N, None)
    for _ in range(3):
        psi.copy_(start)
        P.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(torch.view_as_real(psi), torch.view_as_real(want)) and torch.equal(P, wantP)
        gpu_evolve(prec, M, J, dt, steps, 0, seed=9)


@pytest.mark.parametrize("prec", [C128, C64])
@pytest.mark.parametrize("M", [1, 2, 3, 9, 20])
def test_initial_states_and_observable_at_every_kind_of_site(prec, M):
    """Amplitudes to a few roundings of the type, zeros exact, the observable
    of the stored amplitudes to FP64."""
    import torch
    scale = 2.0 ** (-(M - 1) / 2)
    tol = (4 if prec == C128 else 1) * (2.0 ** -53 if prec == C128 else 2.0 ** -24) * scale
    for n in sorted({0, min(1, M - 1), M // 2, M - 1}):
        for product in (False, True):
            note("init", prec, M, n, product)
            psi = torch.full((2 ** M,), float("nan"), dtype=torch_dtype(prec), device="cuda")
            P = torch.zeros(1, dtype=torch.float64, device="cuda")
            (spq.spin_init_product if product else spq.spin_init_random_phase)(psi, M, n, 17)
            got = psi.cpu().numpy().astype(np.complex128)
            up = (np.arange(2 ** M) >> n) & 1 == 0
            if product:
                want = oracle.product_state(M, n, oracle.product_phases(M, 17))
            else:
                # extended precision: the double-precision oracle rounds 2 pi u itself
                turn = 8 * np.arctan(np.longdouble(1)) * oracle.phase_u_array(17, np.arange(2 ** (M - 1))).astype(np.longdouble)
                want = np.zeros(2 ** M, dtype=np.clongdouble)
                want[up] = (np.cos(turn) + 1j * np.sin(turn)) * np.sqrt(np.longdouble(2)) ** -(M - 1)
            assert np.all(got[~up] == 0)
            # a product state sums M - 1 phases here and multiplies M - 1 factors in the oracle
            extra = 4e-15 * M * scale if product else 0.0
            assert np.abs(got - want).max() <= tol + extra
            for site in range(M):
                spq.spin_local_polarization(psi, M, site, P)
                w = np.abs(got) ** 2
                sgn = 1.0 - 2.0 * ((np.arange(2 ** M) >> site) & 1)
                assert abs(float(P[0]) - float((w * sgn).sum())) < 1e-12


@pytest.mark.parametrize("prec", [C128, C64])
def test_batches_of_equal_couplings_share_tables_not_states(prec):
    """Equal couplings with other states, seeds, polarised sites and initial
    kinds, two of them in flight on two streams, against single runs."""
    import torch
    note("batch tables", prec)
    dt, steps = 0.03, 4
    nets = [(9, workloads.ladder(4) + [(0, 8, 0.2, 0.3)]), (15, workloads.star(15, 3)), (17, workloads.star(17, 4)),
            (15, workloads.star(15, 3))]
    spq.spin_release_caches()

    def problems(first):
        return [{"psi": torch.zeros(2 ** M, dtype=torch_dtype(prec), device="cuda"), "M": M, "couplings": J,
                 "observed_site": 1, "polarized_site": (first + q) % M, "seed": first + q,
                 "P": torch.zeros(steps + 1, dtype=torch.float64, device="cuda"),
                 "N": torch.zeros(steps + 1, dtype=torch.float64, device="cuda")} for q, (M, J) in enumerate(nets)]

    calls = [(problems(3), spq.SPIN_INIT_RANDOM_PHASE), (problems(40), spq.SPIN_INIT_RANDOM_PHASE),
             (problems(5), spq.SPIN_INIT_PRODUCT)]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    for k, (ps, init) in enumerate(calls):
        spq.spin_trotter_evolve_batch(ps, prec, dt, steps, init=init, stream=streams[k % 2].cuda_stream)
    torch.cuda.synchronize()
    assert spq.spin_batch_status() == 0
    for ps, init in calls:
        for p in ps:
            psi = torch.empty_like(p["psi"])
            P, N = torch.zeros_like(p["P"]), torch.zeros_like(p["P"])
            make = spq.spin_init_product if init == spq.SPIN_INIT_PRODUCT else spq.spin_init_random_phase
            make(psi, p["M"], p["polarized_site"], p["seed"])
            spq.spin_trotter_evolve_ex(psi, p["M"], p["couplings"], dt, steps, 1, P, N)
            torch.cuda.synchronize()
            assert float((P - p["P"]).abs().max()) < TOL_P[prec]
            assert_state_close(p["psi"].cpu().numpy().astype(np.complex128), psi.cpu().numpy().astype(np.complex128), prec)


def test_default_and_explicit_double_precision_tiles_keep_their_plans():
    """At M = 28, 21 steps, the default takes tiles of 2^14: asking for 2^13
    before or after it changes neither call's bits."""
    import torch
    M, J, dt, steps = 28, workloads.ladder(14), 0.05, 21
    args = (C128, M, J, dt, steps, 0)
    assert [spq.spin_describe_plan(*args, o)["tile_bits"] for o in (spq.Options(), spq.Options(tile_bits=13))] == [14, 13]

    def run(opts):
        note("plans", opts)
        P, N, _, psi = gpu_evolve(C128, M, J, dt, steps, 0, seed=4, opts=opts, keep_state=False)
        return P, N, psi

    def same(a, b):
        return np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]) and torch.equal(a[2], b[2])

    spq.spin_release_caches()
    default = run({})
    spq.spin_release_caches()
    explicit = run({"tile_bits": 13})
    assert not np.array_equal(default[0], explicit[0])
    assert same(run({}), default)                   # after the explicit call
    spq.spin_release_caches()
    run({})
    assert same(run({"tile_bits": 13}), explicit)   # after the default call


@pytest.mark.parametrize("prec,M", [(C64, 13), (C128, 13)])
def test_threads_on_one_stream_do_not_share_partial_sums(prec, M):
    """Dipolar states of 12 to 14 sites run as tiled passes whose partial sums
    lie in the stream's scratch memory: calls of several threads on one stream
    give the bits of calls made one by one."""
    import threading
    import torch
    note("threads", prec, M)
    J = workloads.star(M, 7, a_over_b=-2.0)
    dt, steps, n, calls = 0.03, 6, 4, 12
    spq.spin_prepare_plan(prec, M, J, dt, steps, 0, None)
    psi = [torch.empty(2 ** M, dtype=torch_dtype(prec), device="cuda") for _ in range(n)]
    out = torch.zeros(2, n, calls, steps + 1, dtype=torch.float64, device="cuda")
    norm = torch.zeros_like(out)
    Pall = torch.zeros(2, n, calls, (steps + 1) * M, dtype=torch.float64, device="cuda")
    one = torch.zeros(2, n, calls, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    failed = []

    def work(q, row):
        try:
            for c in range(calls):
                spq.spin_init_random_phase(psi[q], M, 0, 100 * q + c)
                spq.spin_trotter_evolve_ex(psi[q], M, J, dt, steps, 0, out[row, q, c], norm[row, q, c])
                spq.spin_local_polarization(psi[q], M, 0, one[row, q, c:c + 1])
                spq.spin_trotter_evolve_profile(psi[q], M, J, dt, steps, Pall[row, q, c])
        except Exception as e:      # noqa: BLE001 - reported below
            failed.append(e)

    for q in range(n):
        work(q, 0)
    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(q, 1)) for q in range(n)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not failed, failed
    for a in (out, norm, Pall, one):
        assert torch.equal(a[0], a[1])


@pytest.mark.parametrize("prec,M", [(C64, 18), (C64, 24), (C128, 20), (C64, 13)])
def test_autotuner_tries_the_default_first_and_once(prec, M):
    import torch
    torch.zeros(1, device="cuda")
    note("autotune", prec, M)
    J, dt = workloads.ladder(M // 2), 0.05
    spq.spin_release_caches()
    res = spq.spin_autotune(prec, M, J, dt, 0, trial_steps=4)["results"]
    names = ("tile_bits", "reg_bits", "coalesce_bits", "exchange")
    assert all(r["status"] == 0 for r in res) and [res[0][k] for k in names] == [0] * 4
    shapes = [spq.spin_describe_plan(prec, M, J, dt, 4, 0, spq.Options(**{k: r[k] for k in names})) for r in res]
    assert all([s[k] for k in names] != [shapes[0][k] for k in names] for s in shapes[1:])


@pytest.mark.parametrize("prec,M", [(C128, 25), (C128, 26), (C64, 25)])
def test_observable_of_states_around_the_last_level_cache(prec, M):
    """Either way of reading a state against torch's FP64 sums."""
    import torch
    note("observable", prec, M)
    psi = torch.empty(2 ** M, dtype=torch_dtype(prec), device="cuda")
    spq.spin_init_random_phase(psi, M, 3, 8)
    P, N = torch.zeros(1, dtype=torch.float64, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
    w = torch.view_as_real(psi).double().square().sum(-1)
    for site in (0, 1, 3, M - 1):
        spq.spin_local_polarization_ex(psi, M, site, P, N)
        v = w.view(-1, 2, 2 ** site)
        want = float(v[:, 0].sum() - v[:, 1].sum())
        assert abs(float(P) - want) < 1e-12 and abs(float(N) - float(w.sum())) < 1e-12


@pytest.mark.parametrize("prec,M,J,steps", [
    (C64, 20, workloads.star(20, 7), 2), (C64, 21, workloads.star(21, 7), 2),
    (C64, 21, workloads.chain(21, a_over_b=-2.0), 4), (C64, 22, workloads.ladder(11), 4),
    (C64, 23, workloads.chain(23, a_over_b=0.5), 3), (C64, 24, workloads.ladder(12), 3),
    (C128, 20, workloads.ladder(10), 6), (C128, 21, workloads.chain(21), 4), (C128, 22, workloads.ladder(11, a_over_b=0.5), 3),
], ids=lambda v: str(v) if isinstance(v, int) else "")
def test_default_shapes_past_the_smallest_tiles_match_the_oracle(prec, M, J, steps):
    """Tiles of 2^12, 2^13 on 512 lanes (M = 21), and 2^14 with 32 and 64
    amplitudes per lane, where the default goes from one to the next."""
    note("dispatch", M, prec)
    site = M - 1
    ref = np.ascontiguousarray(oracle.random_phase_state(M, site, 5))
    P0, N0 = cref.trotter_run(ref, M, J, 0.03, steps, site)
    P, N, psi, _ = gpu_evolve(prec, M, J, 0.03, steps, site, polarized=site, seed=5)
    assert np.abs(P - P0).max() < TOL_P[prec]
    assert np.abs(N / N0 - 1).max() < TOL_P[prec]
    assert_state_close(psi, ref, prec)


@pytest.mark.parametrize("M", [21, 23])
def test_default_profiles_past_the_smallest_tiles_match_the_single_site_curves(M):
    note("dispatch profile", M)
    J, steps = workloads.chain(M), 5
    Pall, N, _ = gpu_profile(C64, M, J, 0.05, steps, seed=3, keep_state=False)
    for site in (0, M // 2, M - 1):
        P, N1, _, _ = gpu_evolve(C128, M, J, 0.05, steps, site, seed=3, keep_state=False)
        assert np.abs(Pall[:, site] - P).max() < TOL_P[C64]
    assert np.abs(N - N1).max() < TOL_P[C64]
