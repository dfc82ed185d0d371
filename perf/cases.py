"""Performance cases of the random-phase spin-dynamics path.

Each case is one call sequence a user's program makes through the public
entry points, at sizes of this repository's workloads and tests:

* ``evolve``: write the random-phase state, evolve it, keep the polarisation
  curve, the norm curve and the final state;
* ``profile``: the same with the polarisation of every site per step;
* ``batch``: many independent stars of uneven size in one launch;
* ``ensemble``: the ensemble average member by member;
* ``state``: write an initial state and read one site's polarisation, the
  two calls around every evolution.

``prepare`` holds what such a program keeps: the coupling list, device
buffers and the prepared plan.  Curves of complex64 runs are kept in single
precision, the accuracy of the amplitudes they are read from.
"""
import math

import torch

import paper_0710_3747_amd as spin
import workloads

PREC = {"c64": (spin.SPIN_C64, torch.complex64), "c128": (spin.SPIN_C128, torch.complex128)}


def listed():
    return [
        # the 2x5 ladder workload as it stands: the smallest call, one state on one compute unit
        {"name": "ladder_2x5_c64", "kind": "evolve", "net": "ladder", "M": 10, "prec": "c64", "dt": 0.05, "steps": 400},
        # the dipolar star of the Fig. 3(b) check (every pair, I^z I^z phases, 14 sites), its first steps: over all 250
        # the rounding of the single-precision phases adds up to 2.5e-5 of the state, too much to compare two runs by
        {"name": "dipolar_star14_c64", "kind": "evolve", "net": "dipolar", "M": 14, "prec": "c64", "dt": 0.02, "steps": 40},
        # one disorder realisation of the star in double precision, a size between the tested ones
        {"name": "star17_c128", "kind": "evolve", "net": "star", "M": 17, "prec": "c128", "dt": 0.02, "steps": 100},
        # the 2x9 ladder whose random-phase curve is compared with the ensemble
        {"name": "ladder_2x9_c64", "kind": "evolve", "net": "ladder", "M": 18, "prec": "c64", "dt": 0.05, "steps": 200},
        # the 2x12 ladder workload (2000 steps) in chunks of 200: a state the size of the last-level cache
        {"name": "ladder_2x12_c64", "kind": "evolve", "net": "ladder", "M": 24, "prec": "c64", "dt": 0.05, "steps": 200},
        # the all-to-all star workload: many factors per step, ten sweeps of a 2 GiB state per step
        {"name": "star28_c64", "kind": "evolve", "net": "star28", "M": 28, "prec": "c64", "dt": 0.02, "steps": 4},
        # the headline workload, an 8 GiB state, at the benchmark's 20 steps
        {"name": "ladder_2x15_c64", "kind": "evolve", "net": "ladder", "M": 30, "prec": "c64", "dt": 0.05, "steps": 20},
        # the same state in double precision (16 GiB): the reference run of the precision comparison
        {"name": "ladder_2x15_c128", "kind": "evolve", "net": "ladder", "M": 30, "prec": "c128", "dt": 0.05, "steps": 5},
        # polarisation profile of every site of a 2x13 ladder
        {"name": "profile_2x13_c64", "kind": "profile", "net": "ladder", "M": 26, "prec": "c64", "dt": 0.05, "steps": 50},
        # disorder average: stars of 14..20 sites, as the batch workload draws them
        {"name": "batch_stars_c64", "kind": "batch", "n": 32, "m_lo": 14, "m_hi": 20, "prec": "c64", "dt": 0.02, "steps": 25},
        # the whole 14-site ensemble member by member (8192 members in one stacked evolution)
        {"name": "ensemble_2x7_c64", "kind": "ensemble", "net": "ladder", "M": 14, "prec": "c64", "dt": 0.05, "steps": 50},
        # initial state and its polarisation alone, as a program does that draws states and measures them
        {"name": "state28_c64", "kind": "state", "init": "random", "M": 28, "site": 0, "prec": "c64"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["evolve"] * 6 + ["profile", "batch", "ensemble", "state"])
    prec = rng.choice(["c64", "c64", "c128"])
    if kind == "state":
        M = rng.randint(12, 28)
        return {"kind": kind, "init": rng.choice(["random", "random", "product"]), "M": M, "site": rng.randrange(M), "prec": prec}
    if kind == "batch":
        lo = rng.randint(8, 16)
        return {"kind": kind, "n": _log(rng, 4, 32), "m_lo": lo, "m_hi": min(20, lo + rng.randint(0, 5)), "prec": prec, "dt": 0.02,
                "steps": _log(rng, 3, 25)}
    if kind == "ensemble":
        return {"kind": kind, "net": rng.choice(["ladder", "star", "chain"]), "M": rng.randint(9, 13), "prec": prec, "dt": 0.05,
                "steps": _log(rng, 5, 50)}
    net = rng.choice(["ladder", "ladder", "chain", "star", "dipolar"])
    dense = net in ("star", "dipolar")
    M = rng.randint(8, 24 if dense else 27)
    if net == "ladder":
        M -= M % 2
    # long runs of small states, short runs of large ones
    most = max(3, min(400, 2 ** (29 - M) if dense else 2 ** (33 - M)))
    if net in ("chain", "dipolar"):
        # I^z I^z phases: single-precision rounding grows with the number of factors (see the listed dipolar star)
        most = max(3, min(most, 7500 // (M * (M - 1) if dense else 2 * M)))
    return {"kind": kind, "net": net, "M": M, "prec": prec, "dt": 0.02 if dense else 0.05, "steps": _log(rng, max(2, most // 16), most)}


def _couplings(case):
    net, M = case["net"], case["M"]
    if net == "ladder":
        return workloads.ladder(M // 2)
    if net == "chain":
        return workloads.chain(M, a_over_b=0.5)
    if net == "star28":
        return workloads.star_m28()
    if net == "star":
        return workloads.star(M, 2000 + M)
    return workloads.star(M, 77, 1.0, 1.0, a_over_b=-2.0)


def _problems(case):
    return workloads.star_batch(case["n"], case["m_lo"], case["m_hi"], 4, 2000, 1000)


def prepare(case, seed):
    prec, dtype = PREC[case["prec"]]
    kind = case["kind"]
    f64 = dict(dtype=torch.float64, device="cuda")
    s = {"case": case, "kind": kind, "prec": prec, "seed": seed}
    if kind == "state":
        s.update(psi=torch.empty(2 ** case["M"], dtype=dtype, device="cuda"), P=torch.empty(1, **f64), N=torch.empty(1, **f64))
        return s
    rows = case["steps"] + 1
    if kind == "batch":
        problems = _problems(case)
        s["psi"] = torch.empty(sum(2 ** p["M"] for p in problems), dtype=dtype, device="cuda")
        s["P"], s["N"] = (torch.empty(len(problems), rows, **f64) for _ in range(2))
        states = s["psi"].split([2 ** p["M"] for p in problems])
        s["problems"] = [
            {"psi": states[r], "M": p["M"], "couplings": p["couplings"], "observed_site": 0, "polarized_site": 0, "seed": seed * 4096 + r,
             "P": s["P"][r], "N": s["N"][r]}
            for r, p in enumerate(problems)
        ]
        return s
    M, J = case["M"], _couplings(case)
    s.update(J=J, N=torch.empty(rows, **f64))
    if kind == "ensemble":
        # members of one evolution fill this buffer; a contiguous range of them is averaged
        s["work"] = torch.empty(2 ** (2 * M - 1), dtype=dtype, device="cuda")
        s["first"] = seed % 997
        s["P"] = torch.empty(rows, **f64)
        return s
    s["psi"] = torch.empty(2 ** M, dtype=dtype, device="cuda")
    s["P"] = torch.empty(rows * (M if kind == "profile" else 1), **f64)
    spin.spin_prepare_plan(prec, M, J, case["dt"], case["steps"], spin.SPIN_ALL_SITES if kind == "profile" else 0)
    return s


def _kept(s, *curves):
    return [c.to(torch.float32) if s["prec"] == spin.SPIN_C64 else c for c in curves]


def run(s):
    case, kind = s["case"], s["kind"]
    if kind == "state":
        init = spin.spin_init_product if case["init"] == "product" else spin.spin_init_random_phase
        init(s["psi"], case["M"], case["site"], s["seed"])
        spin.spin_local_polarization_ex(s["psi"], case["M"], case["site"], s["P"], s["N"])
        return {"psi": s["psi"], "P": s["P"], "N": s["N"]}
    if kind == "batch":
        spin.spin_trotter_evolve_batch(s["problems"], s["prec"], case["dt"], case["steps"])
        P, N = _kept(s, s["P"], s["N"])
        return {"psi": s["psi"], "P": P, "N": N}
    if kind == "ensemble":
        spin.spin_ensemble_evolve(s["work"], case["M"], s["J"], case["dt"], case["steps"], 0, 0, s["P"], s["N"],
                                  first_member=s["first"], n_members=2 ** (case["M"] - 1) - s["first"])
        P, N = _kept(s, s["P"], s["N"])
        return {"P": P, "N": N}
    spin.spin_init_random_phase(s["psi"], case["M"], 0, s["seed"])
    if kind == "profile":
        spin.spin_trotter_evolve_profile(s["psi"], case["M"], s["J"], case["dt"], case["steps"], s["P"], s["N"])
    else:
        spin.spin_trotter_evolve(s["psi"], case["M"], s["J"], case["dt"], case["steps"], 0, s["P"], s["N"])
    P, N = _kept(s, s["P"], s["N"])
    return {"psi": s["psi"], "P": P, "N": N}


def _factors(K, steps):
    """Two-spin factors of `steps` steps; the two halves of a step share the last coupling's factor."""
    return (2 * K - 1) * steps if K else 0


def work(case):
    """Bytes of the outputs, each written once, and 12 flops per anti-aligned amplitude pair and factor."""
    size = 8 if case["prec"] == "c64" else 16
    if case["kind"] == "state":
        return {"bytes": size * 2 ** case["M"], "flops": 0}
    rows = 16 * (case["steps"] + 1)
    if case["kind"] == "batch":
        Ms = [p["M"] for p in _problems(case)]
        return {"bytes": sum(size * 2 ** M + rows for M in Ms),
                "flops": sum(3 * 2 ** M * _factors(M * (M - 1) // 2, case["steps"]) for M in Ms)}
    M = case["M"]
    if case["kind"] == "profile":
        rows *= (M + 1) // 2
    amps = 2 ** (2 * M - 1) if case["kind"] == "ensemble" else 2 ** M
    return {"bytes": rows if case["kind"] == "ensemble" else size * amps + rows, "flops": 3 * amps * _factors(len(_couplings(case)), case["steps"])}


# ------------------------------------------------------------- plain torch in 64 bits

def _uniform(seed, r):
    """Output r+1 of the SplitMix64 stream `seed` (wrapping int64 arithmetic) as a uniform in [0, 1)."""
    def signed(v):
        v &= 2 ** 64 - 1
        return v - 2 ** 64 if v >= 2 ** 63 else v

    def shr(z, n):
        return (z >> n) & (2 ** (64 - n) - 1)

    z = (r + 1) * signed(0x9E3779B97F4A7C15) + signed(seed)
    z = (z ^ shr(z, 30)) * signed(0xBF58476D1CE4E5B9)
    z = (z ^ shr(z, 27)) * signed(0x94D049BB133111EB)
    z = z ^ shr(z, 31)
    return shr(z, 11).to(torch.float64) * 2.0 ** -53


def _exact_state(M, site, seed, product=False):
    psi = torch.zeros(2 ** M, dtype=torch.complex128, device="cuda")
    up = psi.view(2 ** (M - 1 - site), 2, 2 ** site)[:, 0, :]
    r = torch.arange(2 ** (M - 1), device="cuda")
    if product:
        u = _uniform(seed, torch.arange(M, device="cuda"))
        phase = torch.zeros(2 ** (M - 1), dtype=torch.float64, device="cuda")
        for q, l in enumerate(l for l in range(M) if l != site):
            phase -= u[l] * (1 - ((r >> q) & 1)).to(torch.float64)
    else:
        phase = _uniform(seed, r)
    phase = 2 * math.pi * (phase - torch.floor(phase))
    up.copy_(torch.polar(torch.full_like(phase, 2.0 ** (-(M - 1) / 2)), phase).view(up.shape))
    return psi


def _pair(psi, i, j):
    lo, hi = min(i, j), max(i, j)
    return psi.view(-1, 2, 2 ** (hi - lo - 1), 2, 2 ** lo)


def _exact_factor(psi, i, j, A, B):
    v = _pair(psi, i, j)
    x, y = v[:, 0, :, 1], v[:, 1, :, 0]
    ph = complex(math.cos(A / 4), math.sin(A / 4))
    c, s = math.cos(B / 2) * ph, -1j * math.sin(B / 2) * ph
    old = x.clone()
    x.mul_(c).add_(y, alpha=s)
    y.mul_(c).add_(old, alpha=s)
    if A:
        v[:, 0, :, 0].mul_(ph.conjugate())
        v[:, 1, :, 1].mul_(ph.conjugate())


def _weights(psi, site):
    return torch.view_as_real(psi).view(-1, 2, 2 ** (site + 1)).square().sum(dim=(0, 2))


def _exact_evolve(psi, J, dt, steps, sites):
    order = []
    for i, j, a, b in list(J) + list(J)[::-1]:
        if order and order[-1][:2] == (i, j):
            order[-1] = (i, j, order[-1][2] + a * dt / 2, order[-1][3] + b * dt / 2)
        else:
            order.append((i, j, a * dt / 2, b * dt / 2))
    P, N = [], []
    for k in range(steps + 1):
        if k:
            for i, j, A, B in order:
                _exact_factor(psi, i, j, A, B)
        for site in sites:
            w = _weights(psi, site)
            P.append(w[0] - w[1])
        N.append(w[0] + w[1])
    return torch.stack(P), torch.stack(N)


def _too_long(amps, factors, problems=1):
    """Whether the plain evolution takes over about 20 seconds: sweeps of the state, or many small calls."""
    return factors * (amps * 1.4e-11 + 1.2e-4) * problems > 16.0


def exact(case, seed):
    kind = case["kind"]
    if kind == "state":
        psi = _exact_state(case["M"], case["site"], seed, case["init"] == "product")
        w = _weights(psi, case["site"])
        return {"psi": psi, "P": (w[0] - w[1]).view(1), "N": (w[0] + w[1]).view(1)}
    steps, dt = case["steps"], case["dt"]
    if kind == "batch":
        problems = _problems(case)
        if sum(_factors(len(p["couplings"]), steps) for p in problems) > 2.5e5:
            return None
        out = []
        for r, p in enumerate(problems):
            psi = _exact_state(p["M"], 0, seed * 4096 + r)
            out.append((psi, *_exact_evolve(psi, p["couplings"], dt, steps, [0])))
        return {"psi": torch.cat([o[0] for o in out]), "P": torch.stack([o[1] for o in out]), "N": torch.stack([o[2] for o in out])}
    M, J = case["M"], _couplings(case)
    amps = 2 ** (2 * M - 1) if kind == "ensemble" else 2 ** M
    if _too_long(amps, _factors(len(J), steps)):
        return None
    if kind == "ensemble":
        first, members = seed % 997, 2 ** (M - 1) - seed % 997
        psi = torch.zeros(2 ** (M - 1), 2 ** M, dtype=torch.complex128, device="cuda")
        r = torch.arange(members, device="cuda")
        psi[r, (r + first) * 2] = 1.0
        P, N = _exact_evolve(psi.view(-1), J, dt, steps, [0])
        return {"P": P / members, "N": N / members}
    psi = _exact_state(M, 0, seed)
    P, N = _exact_evolve(psi, J, dt, steps, range(M) if kind == "profile" else [0])
    return {"psi": psi, "P": P, "N": N}
