"""Measured workloads: what a program that uses the library has it do.

Each case is a whole call through the public entry points.  A run of population
annealing is one disorder instance, so a program pays for creating the run,
annealing it and reading its results every time: a pass holds all three.  The
sizes are those of the README, the benchmark and the tests (L = 4 ... 24 on the
cubic lattice, L = 32 on the square one, populations of 10^3 ... 5 10^5,
beta_max = 5, N_S = 10), with shorter schedules for the largest populations.

Kinds:
  run         Pamc(...).anneal(), its observables, overlap histogram and, for
              smaller populations, the final population
  checkpoint  half of a run, its population to the host, and the rest of the
              run from there in a fresh handle
  batch       many instances of mixed size annealed together
  serve       a burst of requests through a standing server
"""
import math
import random

import numpy as np

from paper_1710_09025_amd import Pamc, PamcBatch, PamcServer, default_capacity, make_pm_j

BETA_MAX = 5.0
NAMES = ("R", "sum_E", "E_min", "E_max", "mean_E", "C_V", "lnZ", "S_f", "rho_s", "q_abs", "q2", "q4")
WHOLE = ("R", "sum_E", "E_min", "E_max")

# What one case may hold; a listed or drawn case sets the ones that differ.
DEFAULTS = {"kind": "run", "model": "pm", "dim": 3, "L": 4, "R": 1000, "temps": 101, "sweeps": 10,
            "schedule": "linear", "packed": False, "icm": 0, "overlaps": 1, "population": False,
            "pop_schedule": False, "autotune": False, "instances": 1, "L_min": 4, "L_max": 12}


def _case(name=None, **kw):
    c = dict(DEFAULTS, **kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call in use: a student's first run, an instance of a
        # disorder average over small systems; bound by launches and latency
        _case("run_L4_R1000", L=4, R=1000, temps=101, population=True),
        # the ordinary single instance of the benchmark, tuned shape
        _case("run_L8_R100000", L=8, R=100_000, temps=201, autotune=True),
        # odd lattice, ragged population, overlaps along the way
        _case("run_L13_R30001", L=13, R=30_001, temps=101, overlaps=11),
        # one bit per spin and the LBLT schedule at a size without power of two
        _case("run_L12_packed_lblt", L=12, R=100_000, temps=61, packed=True, schedule="lblt"),
        # the benchmark's largest population, on a third of its temperatures
        _case("run_L16_R500000", L=16, R=500_000, temps=101, autotune=True),
        # a lattice beyond the colour-major layouts
        _case("run_L24_R4000", L=24, R=4000, temps=41),
        # Gaussian couplings, the paper's case study, at the benchmark's size
        _case("gauss_L8_R100000", model="gauss", L=8, R=100_000, temps=101, autotune=True),
        # Gaussian couplings on an odd lattice with a population schedule
        _case("gauss_L9_R20011_pop", model="gauss", L=9, R=20_011, temps=101, pop_schedule=True, population=True),
        # the square lattice with the paper's two cluster-move rounds a step
        _case("square_L32_icm2", model="gauss", dim=2, L=32, R=50_000, temps=61, icm=2),
        # a run interrupted, stored and resumed
        _case("checkpoint_L10_R20000", kind="checkpoint", L=10, R=20_000, temps=101),
        # disorder average: many instances of mixed size as one batch
        _case("batch_mixed_L4_12", kind="batch", instances=64, R=10_000, temps=101, autotune=True),
        # a burst of requests of mixed size on a standing server
        _case("serve_mixed_L4_14", kind="serve", instances=24, R=20_000, temps=101, L_min=4, L_max=14, autotune=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: sizes spread over their logarithm,
    odd ones among them, cut to a fraction of the largest listed one."""
    kind = rng.choice(["run"] * 6 + ["checkpoint", "batch", "serve"])
    temps = rng.randint(21, 151)
    sweeps = rng.choice([10, 10, 10, 5, 7, 20])
    autotune = False
    if kind in ("batch", "serve"):
        hi = rng.randint(8, 14)
        return _case(kind=kind, instances=rng.randint(5, 40), R=_log(rng, 2000, 20_000), temps=temps,
                     sweeps=sweeps, L_min=4, L_max=hi, packed=rng.random() < 0.25,
                     model=rng.choice(["pm", "pm", "gauss"]))
    model = rng.choice(["pm", "pm", "pm", "gauss", "square"])
    icm = rng.choice([0, 0, 0, 1, 2])
    if model == "square":
        dim, L, cost = 2, _log(rng, 8, 64), 4.0
    elif model == "gauss":
        dim, L, cost = 3, _log(rng, 4, 16), 4.0
    else:
        dim, L = 3, _log(rng, 4, 32)
        cost = 1.0 if L < 22 else 8.0
    N = L ** dim
    # at most a twentieth of the largest listed case's attempts
    most = 1e11 / (cost * N * temps * sweeps)
    R = max(50, _log(rng, 200, max(400, min(300_000, most))))
    packed = icm == 0 and rng.random() < 0.25
    small = R * N <= 20_000_000
    return _case(kind=kind, model="pm" if model == "pm" else "gauss", dim=dim, L=L, R=R, temps=temps, sweeps=sweeps,
                 schedule=rng.choice(["linear", "linear", "lblt"]), packed=packed, icm=icm,
                 overlaps=rng.choice([1, 1, 5]), population=small and rng.random() < 0.5,
                 pop_schedule=rng.random() < 0.2)


def _beta(c):
    n = c["temps"]
    if c["schedule"] == "lblt":  # linear in beta up to T = 1, then linear in T
        k = (n - 1) // 2
        up = np.array([j / k for j in range(k)])
        return np.concatenate([up, 1.0 / np.linspace(1.0, 1.0 / BETA_MAX, n - k)])
    return np.array([BETA_MAX * k / (n - 1) for k in range(n)])


def _pop(c, beta):
    """Fewer replicas at low temperature; the first entry is R."""
    if not c["pop_schedule"]:
        return None
    f = 0.25 + 0.75 / (1.0 + np.exp(4.0 * (beta - 1.5)))
    p = np.maximum(1, np.rint(c["R"] * f / f[0])).astype(np.int64)
    p[0] = c["R"]
    return p


def _rows_max(c, pop):
    return c["R"] if pop is None else int(pop.max())


def _couplings(c, L, seed):
    if c["model"] == "pm":
        return make_pm_j(L, seed)
    n = (3, L ** 3) if c["dim"] == 3 else (2, L ** 2)
    j = np.rint(np.random.default_rng(seed).standard_normal(n) * 2.0 ** 20)
    return np.clip(j, -(2 ** 23) + 1, 2 ** 23 - 1).astype(np.int32)


def _instances(c, seed):
    """The sizes of a batch or a burst: L in turn over its range."""
    rng = random.Random(seed)
    beta = _beta(c)
    out = []
    for i in range(c["instances"]):
        L = c["L_min"] + i % (c["L_max"] - c["L_min"] + 1)
        if c["kind"] == "serve":
            R = max(100, int(c["R"] * (0.25 + 1.5 * ((i * 7) % 11) / 10.0)))
        else:
            R = c["R"]
        out.append({"L": L, "couplings": _couplings(c, L, rng.getrandbits(40)), "R": R, "beta": beta,
                    "sweeps": c["sweeps"], "seed": rng.getrandbits(63)})
    return out


def prepare(case, seed):
    c = dict(DEFAULTS, **case)
    if c["kind"] == "batch":
        return {"case": c, "instances": _instances(c, seed)}
    if c["kind"] == "serve":
        server = PamcServer(4 << 30, autotune=c["autotune"], packed=c["packed"])
        return {"case": c, "requests": _instances(c, seed), "server": server}
    beta = _beta(c)
    steps = np.unique(np.linspace(0, c["temps"] - 1, c["overlaps"] + 1).astype(np.int32)[1:])
    rng = random.Random(seed)
    return {"case": c, "couplings": _couplings(c, c["L"], rng.getrandbits(40)), "beta": beta,
            "seed": rng.getrandbits(63), "steps": steps, "pop": _pop(c, beta)}


def _new_run(s):
    c = s["case"]
    return Pamc(c["L"], s["couplings"], c["R"], s["beta"], c["sweeps"], s["seed"], overlap_steps=s["steps"],
                packed=c["packed"], pop_schedule=s["pop"], icm_rounds=c["icm"], autotune=c["autotune"])


def _observed(o):
    return {k: np.asarray(o[k], dtype=np.int64 if k in WHOLE else np.float64) for k in NAMES}


def _population(st, R_max):
    """The population in buffers of the run's capacity, zero beyond its rows."""
    cap = default_capacity(R_max)

    def whole(a):
        out = np.zeros((cap,) + a.shape[1:], dtype=np.int64 if a.dtype == np.uint32 else a.dtype)
        out[: len(a)] = a
        return out

    return {"rows": int(st["R"]), "spins": whole(st["spins"]), "E": whole(st["E"]), "family": whole(st["family"])}


def _check(status):
    if status != 0:
        raise RuntimeError(f"anneal: status {status}")


def _run_one(s):
    with _new_run(s) as p:
        _check(p.anneal())
        out = _observed(p.observables())
        out["overlap"] = np.stack([p.overlap_hist(int(k)) for k in s["steps"]])
        if s["case"]["population"]:
            out.update(_population(p.get_state(), _rows_max(s["case"], s["pop"])))
    return out


def _run_checkpoint(s):
    with _new_run(s) as p:
        _check(p.anneal(s["case"]["temps"] // 2))
        first = _observed(p.observables())
        st = p.get_state()
    with _new_run(s) as p:
        p.set_state(st["step"], st["spins"], st["family"], st["lnZ"])
        _check(p.anneal())
        last = _observed(p.observables())
    return {"first": first, "stored": _population(st, _rows_max(s["case"], s["pop"])), "last": last}


def _stacked(per_instance):
    return {k: np.stack([o[k] for o in per_instance]) for k in NAMES}


def _run_batch(s):
    c = s["case"]
    b = PamcBatch(s["instances"], packed=c["packed"], autotune=c["autotune"])
    try:
        _check(b.anneal())
        return _stacked([_observed(b.observables(i)) for i in range(c["instances"])])
    finally:
        b.close()


def _run_serve(s):
    srv = s["server"]
    ids = [srv.submit(d["L"], d["couplings"], d["R"], d["beta"], d["sweeps"], d["seed"]) for d in s["requests"]]
    out = []
    for rid in ids:
        status, obs, _ = srv.wait(rid, timeout=60.0, interval=0.0005)
        _check(status)
        out.append(_observed(obs))
    return _stacked(out)


def run(state):
    return {"run": _run_one, "checkpoint": _run_checkpoint, "batch": _run_batch,
            "serve": _run_serve}[state["case"]["kind"]](state)


def _attempts(c):
    """Spin-flip attempts of a pass (the population stays near its target)."""
    steps = c["temps"] * c["sweeps"]
    if c["kind"] in ("batch", "serve"):
        return sum(d["R"] * d["L"] ** 3 for d in _instances(dict(c, model="pm"), 0)) * steps
    pop = _pop(c, _beta(c))
    R = float(np.mean(pop)) if pop is not None else float(c["R"])
    return R * c["L"] ** c["dim"] * steps


def work(case):
    """Operations: one draw, one local field and one decision per attempt
    (15.75 32-bit operations with +-1 couplings; 47.5 with real ones, 43 on
    the square lattice).  Bytes: the population, one bit per spin, read and
    written once per temperature."""
    c = dict(DEFAULTS, **case)
    ops = 15.75 if c["model"] == "pm" else (47.5 if c["dim"] == 3 else 43.0)
    att = _attempts(c)
    return {"bytes": att / c["sweeps"] / 8 * 2, "flops": att * ops}


# --- the method once more in plain numpy, for the smallest runs -----------------

def _philox(x, y, z, w, key):
    """Philox4x32-10 of counters (x, y, z, w): four uint32 words."""
    m = np.uint64(0xFFFFFFFF)
    x, y, z, w = (np.asarray(v, dtype=np.uint64) for v in (x, y, z, w))
    k0, k1 = np.uint64(key & 0xFFFFFFFF), np.uint64(key >> 32)
    for _ in range(10):
        a, b = x * np.uint64(0xD2511F53), z * np.uint64(0xCD9E8D57)
        x, y, z, w = (b >> np.uint64(32)) ^ y ^ k0, b & m, (a >> np.uint64(32)) ^ w ^ k1, a & m
        k0, k1 = (k0 + np.uint64(0x9E3779B9)) & m, (k1 + np.uint64(0xBB67AE85)) & m
    return x, y, z, w


def _words(block, row, step, tag, key):
    """[rows][4 blocks] words of the draws of blocks 0 ... for each row."""
    b, r = np.broadcast_arrays(block[None, :], row[:, None])
    return np.stack(_philox(b, r, step, tag, key), axis=-1).reshape(len(row), -1)


def exact(case, seed):
    """The run in plain numpy: +-1 couplings, cubic lattice, small runs."""
    c = dict(DEFAULTS, **case)
    if c["kind"] != "run" or c["model"] != "pm" or c["icm"] or _attempts(c) > 1.5e8:
        return None
    s = prepare(dict(c, autotune=False), seed)
    L, beta, key, T = c["L"], s["beta"], s["seed"], c["temps"]
    N, R = L ** 3, c["R"]
    pop = s["pop"] if s["pop"] is not None else np.full(T, R)
    J = s["couplings"].reshape(3, N).astype(np.int32)
    site = np.arange(N)
    xyz = [site % L, site // L % L, site // L ** 2]
    at = lambda v: v[0] % L + L * (v[1] % L + L * (v[2] % L))  # noqa: E731
    step = [[(q + 1 if i == d else q) for i, q in enumerate(xyz)] for d in range(3)]
    back = [[(q - 1 if i == d else q) for i, q in enumerate(xyz)] for d in range(3)]
    up, down = [at(v) for v in step], [at(v) for v in back]
    if L % 2 == 0:
        colour, ncol = sum(xyz) % 2, 2
    else:
        colour, ncol = sum(np.where(q == L - 1, 2, q % 2) for q in xyz) % 3, 3
    sites = [site[colour == q] for q in range(ncol)]
    w = _words(np.arange((N + 3) // 4), np.arange(R), 0, 0x10000000, key)[:, :N]
    S = np.where(w >> np.uint64(31), 1, -1).astype(np.int32)
    fam = np.arange(R)
    lnZ = N * math.log(2.0)
    out = {k: np.full(T, np.nan) for k in NAMES}
    for k in WHOLE:
        out[k] = np.zeros(T, dtype=np.int64)
    hists = []
    for k in range(T):
        n = len(S)
        rows = np.arange(n)
        thr = [min(int(math.floor(math.exp(-beta[k] * 4.0 * q) * 2.0 ** 32)), 2 ** 32 - 1) for q in (1, 2, 3)]
        table = np.array([2 ** 32] * 4 + thr, dtype=np.uint64)  # by dE / 4 + 3
        for t in range(c["sweeps"]):
            for q, at_q in enumerate(sites):
                h = sum(J[d][at_q] * S[:, up[d][at_q]] + J[d][down[d][at_q]] * S[:, down[d][at_q]] for d in range(3))
                dE = 2 * S[:, at_q] * h
                if beta[k] == 0.0:
                    S[:, at_q] *= -1
                    continue
                blocks = np.arange((len(at_q) + 3) // 4) + (q << 24)
                u = _words(blocks, rows, k, 0x20000000 | t, key)[:, :len(at_q)]
                S[:, at_q] *= np.where(u < table[dE // 4 + 3], -1, 1)
        E = -sum((J[d] * S * S[:, up[d]]).sum(axis=1) for d in range(3)).astype(np.int64)
        counts = np.bincount(fam)
        counts = counts[counts > 0].astype(np.float64)
        S_f = math.log(n) - float(np.sum(counts * np.log(counts))) / n
        mean = float(E.sum()) / n
        var = float(n * int((E * E).sum()) - int(E.sum()) ** 2) / float(n) ** 2
        for name, v in (("R", n), ("sum_E", E.sum()), ("E_min", E.min()), ("E_max", E.max()), ("mean_E", mean),
                        ("C_V", beta[k] ** 2 * var / N), ("lnZ", lnZ), ("S_f", S_f), ("rho_s", n / math.exp(S_f))):
            out[name][k] = v
        if k in s["steps"]:
            Q = (S[: n // 2] * S[n // 2: 2 * (n // 2)]).sum(axis=1)
            hists.append(np.bincount(Q + N, minlength=2 * N + 1).astype(np.int64))
            qq = Q / N
            out["q_abs"][k], out["q2"][k], out["q4"][k] = np.abs(qq).mean(), (qq ** 2).mean(), (qq ** 4).mean()
        if k < T - 1:
            db = beta[k + 1] - beta[k]
            wt = np.exp(-db * (E - E.min()))
            lnZ += -db * float(E.min()) + math.log(float(wt.sum())) - math.log(n)
            tau = pop[k + 1] * wt / wt.sum()
            u = _philox(np.zeros(n), rows, k, 0x30000000, key)[0]
            take = np.floor(tau) + (u < np.floor((tau - np.floor(tau)) * 2.0 ** 32).astype(np.uint64))
            keep = np.repeat(rows, take.astype(np.int64))
            S, fam = S[keep], fam[keep]
    out["overlap"] = np.stack(hists)
    if c["population"]:
        st = {"R": len(S), "spins": S.astype(np.int8), "E": E.astype(np.int32), "family": fam}
        out.update(_population(st, _rows_max(c, s["pop"])))
    return out
