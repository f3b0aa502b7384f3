"""The work that users of this library have it do, as cases to be timed.

A case is one call sequence of a program that uses the library through its
Python entry points (``Lattice``, ``Lattice9``, ``Server``), over sizes from a
lattice of a hundred sites, where a step is all launches and latency, to 2^27
sites, where it is all memory.  The workloads are the paper's experiments at
their own sizes and the larger ones that the benchmark and the tests name.

``prepare`` builds the context (the library writes the Poisson start on the
GPU) and the caller's result buffers; ``run`` is one pass: the steps and the
observables a program asks for after them.  A pass starts from the state the
last one left, as it does in a program.  Every output is whole numbers: the
lattice's counts, moment sums and histograms.
"""
import math

import numpy as np
import torch

from paper_1706_01094_amd.mclg import (FLAG_GALILEAN, FLAG_NO_STREAM, LAMBDA9_PAPER, Lattice, Lattice9,
                                       Server)

MOMENT_WORDS = 33  # int64 values of one moments record
PAD = 128          # the state's arrays are padded to this many counts


def listed():
    return [
        # The smallest runs: one lattice of the paper's size, many steps.
        d1q3("plain_256", n=1, L=256, rho=10, u=0.0, steps=1000),
        # The equilibrium figure: 19 lattices of 100 sites, one per velocity,
        # sampled every ten steps by a host loop.
        d1q3("equilibrium_19x100", n=19, L=100, rho=36, u=0.9, steps=10, mode="sample"),
        # The relaxation figure: a thousand lattices of a thousand sites with
        # 300 particles per site, the moments recorded after every step.
        d1q3("relaxation_1000x1000", n=1000, L=1000, rho=300, u=0.0, steps=1, logs=10, mode="log",
             start="uniform", n_max=300),
        # An ordinary lattice of an odd size, stepped as the library does it
        # by default.
        d1q3("plain_1000003", n=1, L=1_000_003, rho=30, u=0.05, steps=64),
        # A density wave with one Fourier mode recorded every ten steps,
        # several steps per launch.
        d1q3("wave_4M_log10", n=1, L=1 << 22, rho=40, u=0.0, steps=10, logs=25, modes=1, blocked=250,
             mode="log", start="wave"),
        # The benchmark's lattice, by default and with several steps per launch.
        d1q3("plain_16M", n=1, L=1 << 24, rho=50, u=0.1, steps=64),
        d1q3("plain_16M_blocked", n=1, L=1 << 24, rho=50, u=0.1, steps=256, blocked=256),
        # A lattice larger than the caches.
        d1q3("plain_128M", n=1, L=1 << 27, rho=50, u=0.1, steps=16),
        # Many independent lattices of uneven size and density in one context.
        d1q3("replicas_1024", n=1024, L=1 << 18, L_lo=1 << 10, rho=100, rho_lo=5, u=0.2, steps=16),
        # Jobs of uneven size and length through the continuous-batching
        # server, from submission to the last result.
        {"name": "served_48", "kind": "server", "jobs": 48, "L_lo": 1 << 12, "L": 1 << 20,
         "steps_lo": 50, "steps": 250, "rho_lo": 5, "rho": 100, "tick": 50, "sizes_seed": 5},
        # Two dimensions: the equilibrium figure's 13 lattices, sampled by a
        # host loop, and the benchmark's large lattice.
        d2q9("d2q9_13x100x10", n=13, Lx=100, Ly=10, rho=36, ux=0.6, uy=0.25, steps=10, mode="sample"),
        d2q9("d2q9_4096x4096", n=1, Lx=4096, Ly=4096, rho=36, ux=0.0, uy=0.0, steps=4),
    ]


def d1q3(name, *, n, L, rho, u, steps, L_lo=0, rho_lo=0, logs=0, modes=0, blocked=0, bins=0, C=10,
         n_max=255, no_stream=False, galilean=False, mode="step", start="poisson", sizes_seed=4):
    """n lattices of L sites (of L_lo .. L with L_lo), density rho (rho_lo ..
    rho) and velocities spread over -u .. u (u itself for one lattice)."""
    return {"name": name, "kind": "d1q3", "n": n, "L": L, "L_lo": L_lo, "rho": rho, "rho_lo": rho_lo,
            "u": u, "steps": steps, "logs": logs, "modes": modes, "blocked": blocked, "bins": bins,
            "C": C, "n_max": n_max, "no_stream": no_stream, "galilean": galilean, "mode": mode, "start": start,
            "sizes_seed": sizes_seed}


def d2q9(name, *, n, Lx, Ly, rho, ux, uy, steps, C=10, bins=0, mode="step"):
    """n lattices of Lx x Ly sites, x velocities spread over -ux .. ux."""
    return {"name": name, "kind": "d2q9", "n": n, "Lx": Lx, "Ly": Ly, "rho": rho, "ux": ux, "uy": uy,
            "steps": steps, "C": C, "bins": bins, "mode": mode}


def _log_int(rng, lo, hi):
    """A whole number, even over the logarithm of lo .. hi."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["plain", "plain", "blocked", "replicas", "replicas", "log", "histogram",
                       "sample", "d2q9", "d2q9", "server"])
    rho = rng.randint(5, 100)
    u = round(rng.uniform(0.0, 0.2), 3)
    C = rng.choice([10, 10, 10, 5])
    still, galilean = rng.random() < 0.1, rng.random() < 0.07
    if kind == "plain":
        L = _log_int(rng, 64, 1 << 25)
        case = d1q3("", n=1, L=L, rho=rho, u=u, C=C, no_stream=still, galilean=galilean,
                    steps=rng.randint(1, max(1, min(500, (1 << 29) // L))))
    elif kind == "blocked":
        L = 8 * _log_int(rng, 1 << 16, 1 << 21)
        K = rng.randint(8, 128)
        case = d1q3("", n=1, L=L, rho=rho, u=u, C=C, blocked=K, steps=K * rng.randint(1, 2))
    elif kind == "replicas":
        n = _log_int(rng, 2, 256)
        hi = _log_int(rng, 64, min(1 << 18, (1 << 24) // n))
        case = d1q3("", n=n, L=hi, L_lo=rng.choice([max(8, hi // 8), hi]), rho=rho, rho_lo=max(5, rho // 2),
                    u=u, C=C, no_stream=still, galilean=galilean, sizes_seed=rng.randint(0, 1 << 30),
                    steps=rng.randint(1, max(1, min(400, (1 << 28) // (n * hi)))))
    elif kind == "log":
        L = 8 * _log_int(rng, 1 << 13, 1 << 20)
        every, logs = rng.randint(2, 20), rng.randint(2, 20)
        case = d1q3("", n=1, L=L, rho=rho, u=0.0, C=C, steps=every, logs=logs, modes=rng.randint(0, 2),
                    blocked=rng.choice([0, 64]), mode="log", start="wave")
    elif kind in ("histogram", "sample"):
        n = _log_int(rng, 1, 64)
        L = _log_int(rng, 50, 20_000)
        case = d1q3("", n=n, L=L, rho=min(rho, 40), u=u, C=C, steps=rng.randint(1, 25), mode=kind,
                    bins=rng.choice([64, 96, 128]) if kind == "histogram" else 0)
    elif kind == "d2q9":
        Lx, Ly = _log_int(rng, 10, 2048), _log_int(rng, 10, 2048)
        n = _log_int(rng, 1, max(1, min(64, (1 << 21) // (Lx * Ly))))
        mode = rng.choice(["step", "sample", "histogram"])
        case = d2q9("", n=n, Lx=Lx, Ly=Ly, rho=rng.choice([18, 36, 36, 360]), ux=u, uy=round(rng.uniform(0, 0.25), 3),
                    steps=rng.randint(1, 12), mode=mode, bins=64 if mode == "histogram" else 0)
    else:
        case = {"kind": "server", "jobs": rng.randint(4, 32), "L_lo": 1 << 12, "L": _log_int(rng, 1 << 14, 1 << 20),
                "steps_lo": 20, "steps": rng.randint(40, 250), "rho_lo": 5, "rho": rho + 5,
                "tick": rng.choice([25, 50, 100]), "sizes_seed": rng.randint(0, 1 << 30)}
    case.pop("name", None)
    return case


# ---- what a case's sizes are ----------------------------------------------
def _sites(case):
    """Sites of each lattice of a D1Q3 case."""
    n, hi, lo = case["n"], case["L"], case["L_lo"]
    if not lo or lo == hi:
        return np.full(n, hi, dtype=np.uint64)
    g = np.random.Generator(np.random.PCG64(case["sizes_seed"]))
    return g.integers(lo, hi + 1, size=n).astype(np.uint64)


def _laws(case):
    """Density and velocity of each lattice of a D1Q3 case."""
    n = case["n"]
    g = np.random.Generator(np.random.PCG64(case["sizes_seed"] + 1))
    rho = np.full(n, float(case["rho"]))
    if case["rho_lo"]:
        rho = g.integers(case["rho_lo"], case["rho"] + 1, size=n).astype(np.float64)
    u = np.full(n, case["u"]) if n == 1 else np.linspace(-case["u"], case["u"], n)
    return rho, u


def _jobs(case):
    """(job id, sites, steps, density) of a server case."""
    g = np.random.Generator(np.random.PCG64(case["sizes_seed"]))
    jobs = []
    for i in range(case["jobs"]):
        L = int(round(math.exp(g.uniform(math.log(case["L_lo"]), math.log(case["L"])))))
        jobs.append((i, L, int(g.integers(case["steps_lo"], case["steps"] + 1)),
                     float(g.integers(case["rho_lo"], case["rho"] + 1))))
    return jobs


def _zero_padding(state, sites, arrays):
    """Clears the counts between the arrays, which the library never uses, so
    that two states can be compared whole.  Returns the part in use."""
    at, spans = 0, []
    for L in sites:
        stride = -(-int(L) // PAD) * PAD
        for i in range(arrays):
            spans.append(np.arange(at + i * stride + int(L), at + (i + 1) * stride))
        at += arrays * stride
    index = np.concatenate(spans)
    if index.size:
        state.index_fill_(0, torch.from_numpy(index).to(state.device), 0)
    return state[:at]


# ---- inputs -----------------------------------------------------------------
def prepare(case, seed):
    return {"d1q3": _prepare_d1q3, "d2q9": _prepare_d2q9, "server": _prepare_server}[case["kind"]](case, seed)


def _wave(L, rho, seed):
    """Counts [3][L] of a density wave: Poisson of w_i rho (1 + 0.05 sin)."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    x = torch.arange(L, dtype=torch.float64, device="cuda")
    local = (rho * (1.0 + 0.05 * torch.sin(2.0 * math.pi * x / L))).float()
    w = torch.tensor([1 / 6, 2 / 3, 1 / 6], device="cuda")
    return torch.poisson(w[:, None] * local[None, :], generator=g).to(torch.int16)


def _twiddles(L, modes):
    """round(2^24 cos), round(2^24 sin) of 2 pi m x / L, m = 1 .. modes."""
    rows = []
    for m in range(1, modes + 1):
        phase = (torch.arange(L, dtype=torch.int64, device="cuda") * m % L).double() * (2.0 * math.pi / L)
        rows += [torch.round(torch.cos(phase) * (1 << 24)), torch.round(torch.sin(phase) * (1 << 24))]
    return torch.stack(rows).to(torch.int32).contiguous()


def _prepare_d1q3(case, seed):
    sites = _sites(case)
    rho, u = _laws(case)
    kw = {"C": case["C"], "n_max": case["n_max"], 
          "flags": (FLAG_NO_STREAM if case["no_stream"] else 0) | (FLAG_GALILEAN if case["galilean"] else 0)}
    if case["start"] == "poisson":
        kw.update(rho=rho, u0=u)
    elif case["start"] == "wave":
        kw.update(counts=_wave(case["L"], case["rho"], seed))
    else:  # every site the same, a third of the particles at each velocity
        kw.update(counts=torch.full((3 * int(sites.sum()),), case["rho"] // 3, dtype=torch.int16, device="cuda"))
    lat = Lattice(sites, int(seed), **kw)
    if case["blocked"]:
        lat.set_blocked(case["blocked"])
    s = {"case": case, "lattice": lat, "state": _zero_padding(lat.state, sites, 3)}
    if case["mode"] == "log":
        s["log"] = torch.zeros(case["logs"] * case["n"] * MOMENT_WORDS, dtype=torch.int64, device="cuda")
        s["twiddle"] = _twiddles(case["L"], case["modes"]) if case["modes"] else None
    if case["mode"] == "histogram":
        s["histogram"] = torch.zeros((case["n"], 3, case["bins"]), dtype=torch.int64, device="cuda")
    return s


def _prepare_d2q9(case, seed):
    n = case["n"]
    ux = np.full(n, case["ux"]) if n == 1 else np.linspace(-case["ux"], case["ux"], n)
    lat = Lattice9([case["Lx"]] * n, case["Ly"], int(seed), C=case["C"], lams=LAMBDA9_PAPER,
                   rho=np.full(n, float(case["rho"])), ux=ux, uy=np.full(n, case["uy"]))
    s = {"case": case, "lattice": lat, "state": _zero_padding(lat.state, [case["Lx"] * case["Ly"]] * n, 9)}
    if case["mode"] == "histogram":
        s["histogram"] = torch.zeros((n, 9, case["bins"]), dtype=torch.int64, device="cuda")
    return s


def _prepare_server(case, seed):
    jobs = _jobs(case)
    room = sum(6 * (-(-L // PAD) * PAD) for _, L, _, _ in jobs)
    # an arena for half of the jobs at once: the others wait for room
    arena = max(room // 2, max(6 * (L + PAD) for _, L, _, _ in jobs) + 4096)
    return {"case": case, "server": Server(arena, max(2, len(jobs) // 2), int(seed)), "jobs": jobs}


# ---- one pass -----------------------------------------------------------------
def run(s):
    case = s["case"]
    if case["kind"] == "server":
        return _run_server(s)
    lat, mode = s["lattice"], case["mode"]
    if mode == "log":
        lat.step_log(case["steps"], case["logs"], s["log"], s["twiddle"], case["modes"])
        return {"state": s["state"], "log": s["log"]}
    lat.step(case["steps"])
    if mode == "step":
        return {"state": s["state"]}
    if mode == "histogram":
        lat.histogram(case["bins"], s["histogram"])
        return {"state": s["state"], "histogram": s["histogram"]}
    if case["kind"] == "d2q9":
        return {"state": s["state"], "moments": lat.moments_array()}
    records = lat.moments()
    return {"state": s["state"], **{k: np.array([m[k] for m in records]) for k in
                                    ("sum_n", "sum_n2", "sum_nn", "sum_N", "sum_J", "sum_N2", "n0_odd", "max_N")}}


def _run_server(s):
    server, left, results = s["server"], len(s["jobs"]), []
    for job, L, steps, rho in s["jobs"]:
        server.submit(job, L, steps, rho)
    while left:
        server.tick(s["case"]["tick"])
        got = server.poll()
        left -= len(got)
        results += got
    results.sort(key=lambda r: r[0])
    return {"sum_n": np.array([m["sum_n"] for _, m in results]), "sum_n2": np.array([m["sum_n2"] for _, m in results]),
            "sum_nn": np.array([m["sum_nn"] for _, m in results]), "max_N": np.array([m["max_N"] for _, m in results]),
            "digest": np.array([m["digest"] for _, m in results], dtype=np.uint64).view(np.int64)}


# ---- what a pass cannot do without ---------------------------------------------
# Whole-number operations of one site update.  D1Q3: a quarter of a
# Philox4x32-10 call (10 rounds of 2 multiplies and 4 exclusive ors) and the
# draw and update of a site (about 15).  D2Q9: per sub-collision one call and
# about 20 for the pair, the target and the update.
OPS_D1Q3 = 30
OPS_D2Q9 = 80


def work(case):
    """Bytes: the counts read and written once per pass (the steps between
    need no memory), and the observables' own inputs and results."""
    if case["kind"] == "server":
        jobs = _jobs(case)
        # a job starts inside the pass and ends as one record
        return {"bytes": float(sum(6 * L + 8 * MOMENT_WORDS for _, L, _, _ in jobs)),
                "flops": float(OPS_D1Q3 * sum(L * steps for _, L, steps, _ in jobs))}
    if case["kind"] == "d2q9":
        sites = case["n"] * case["Lx"] * case["Ly"]
        extra = {"sample": 8 * 60, "histogram": 16 * 9 * case["bins"], "step": 0}[case["mode"]] * case["n"]
        return {"bytes": float(36 * sites + extra), "flops": float(OPS_D2Q9 * case["C"] * sites * case["steps"])}
    sites = int(_sites(case).sum())
    steps = case["steps"] * max(1, case["logs"])
    extra = {"step": 0, "sample": 8 * MOMENT_WORDS * case["n"], "histogram": 16 * 3 * case["bins"] * case["n"],
             "log": 8 * MOMENT_WORDS * case["n"] * case["logs"] + 8 * case["modes"] * sites}[case["mode"]]
    return {"bytes": float(12 * sites + extra), "flops": float(OPS_D1Q3 * sites * steps)}


def exact(case, seed):
    """The outputs are whole numbers of a stated random sequence: there is no
    64-bit value for them to be near."""
    return None
