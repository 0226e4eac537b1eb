"""Timed cases of the engine: whole calls through the Python entry points.

Three kinds of call are timed, as programs that use the engine make them:

- "run":      a planned simulation (`qew.Simulation`) run from the flat start to
              its horizon with measurements at log-spaced steps, then the
              series, the ensemble averages and, where the case asks for them,
              the final states or the structure factor;
- "critical": `critical.critical_forces`, the bisection for the critical force
              and configuration of periodic samples, from host arrays to host
              arrays;
- "fscan":    `std.fscan`, a scan over drives, with the plan, the workspace and
              the choice of the launch geometry inside the call.

`exact` repeats "run" and "fscan" cases in plain FP64 torch.
"""
import math

import numpy as np
import torch

from paper_1211_7275_amd import critical, qew, std, workloads

RF, RB, RB_LIN, RF_PC = workloads.RF, workloads.RB, workloads.RB_LIN, workloads.RF_PC
C, DT = 1.0, 0.05


def _run_case(name, kind, L, samples, steps, points, f=1.0, fp64=False, k=0, tile=0, drives=1,
              spacing=0.0, uneven_to=0, period=0, sq_bins=0, states=0):
    """L: chain length (with uneven_to: lengths are spread over [L, uneven_to]);
    samples per drive; drives f, f + spacing, ...; k = tile = 0: autotuned;
    sq_bins: -1 for every mode; states: the final configurations of so many samples are
    read back."""
    c = {"call": "run", "kind": kind, "L": L, "samples": samples, "steps": steps, "points": points,
         "f": f, "fp64": fp64, "k": k, "tile": tile, "drives": drives, "spacing": spacing,
         "uneven_to": uneven_to, "period": period, "sq_bins": sq_bins, "states": states}
    if name:
        c["name"] = name
    return c


def _critical_case(name, kind, L, M, samples, tol_f, f_hi=4.0):
    c = {"call": "critical", "kind": kind, "L": L, "M": M, "samples": samples, "tol_f": tol_f,
         "f_hi": f_hi}
    if name:
        c["name"] = name
    return c


def _fscan_case(name, kind, L, drives, f_min, f_max, disorders, steps, points):
    c = {"call": "fscan", "kind": kind, "L": L, "drives": drives, "f_min": f_min, "f_max": f_max,
         "disorders": disorders, "steps": steps, "points": points}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # A small system run to its full horizon (four lines of 1024 sites, 10^4 steps): quick
        # looks, parameter checks and tests.  Few sites per step, so launches and latency count.
        _run_case("small_fp32", RF, 1024, 4, 10_000, 50, states=4),
        # The same in FP64, the reference precision.
        _run_case("small_fp64", RF, 1024, 4, 10_000, 50, fp64=True, states=4),
        # A batch of 512 lines of unequal, odd lengths between 2^10 and 2^16 (finite-size
        # studies), geometry chosen by the autotuner.
        _run_case("uneven_fp32", RF, 1 << 10, 512, 4_000, 60, uneven_to=1 << 16, states=16),
        # Random bond below the threshold, 64 disorders under three drives: lines that pin.
        _run_case("pinned_rb_fp32", RB, 1 << 16, 64, 10_000, 60, f=0.8, drives=3, spacing=0.2,
                  k=96, tile=2048, states=16),
        # The large chain of the benchmark (2^22 sites x 4), in the benchmark's launch geometry,
        # over the first 10^4 steps.
        _run_case("large_fp32", RF, 1 << 22, 4, 10_000, 100, k=56, tile=2048, states=1),
        # The large chain in FP64.
        _run_case("large_fp64", RF, 1 << 22, 4, 1_000, 20, fp64=True, states=1),
        # Paper-scale lines (2^25 sites) under five drives around the random-bond threshold.
        _run_case("paper_rb_fp32", RB, 1 << 25, 1, 500, 16, f=1.897, drives=5, spacing=0.02, k=96,
                  tile=3072),
        # Structure factor of every mode during the relaxation of 64 lines of 8192 sites.
        _run_case("sq_8192_fp32", RF, 8192, 64, 2_000, 30, sq_bins=-1),
        # Structure factor of the large chain in 64 log-spaced bins.
        _run_case("sq_large_fp32", RF, 1 << 22, 4, 400, 30, k=56, tile=2048, sq_bins=64),
        # Critical forces and configurations of a batch of square random-bond samples.
        _critical_case("critical_rb_256", RB, 256, 256, 32, 1e-3),
        # The same for random-field samples of odd length.
        _critical_case("critical_rf_63", RF, 63, 64, 48, 1e-4),
        # Scan over drives for the depinning threshold: the whole analysis call.
        _fscan_case("fscan_rf", RF, 1 << 14, 12, 0.1, 2.0, 2, 4_000, 60),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["fp32", "fp32", "fp64", "fp64", "uneven", "sq", "critical", "critical", "fscan"])
    if family == "critical":
        return _critical_case(None, rng.choice([RF, RB]), _log_int(rng, 17, 257), _log_int(rng, 32, 256),
                              _log_int(rng, 4, 96), rng.choice([1e-2, 1e-3]))
    if family == "fscan":
        f_min = round(rng.uniform(0.05, 0.4), 3)
        return _fscan_case(None, rng.choice([RF, RB]), _log_int(rng, 1_000, 20_000), rng.randint(4, 12),
                           f_min, round(f_min + rng.uniform(1.0, 2.5), 3), rng.randint(1, 3),
                           _log_int(rng, 500, 4_000), rng.randint(20, 60))
    kind = rng.choice([RF, RF, RB, RB, RB_LIN, RF_PC])
    f = round(rng.uniform(0.4, 2.4), 3)
    period = rng.choice([0, 0, 0, _log_int(rng, 16, 4096)])
    if family == "sq":
        L = 1 << rng.randint(8, 20)
        samples = max(1, min(64, _log_int(rng, 1, 64), (1 << 22) // L))
        return _run_case(None, rng.choice([RF, RB]), L, samples, _log_int(rng, 100, 800), rng.randint(5, 30),
                         f=f, fp64=rng.random() < 0.5, period=period,
                         sq_bins=-1 if L <= 1 << 14 else rng.randint(16, 64))
    steps = _log_int(rng, 300, 6_000)
    points = rng.randint(10, 60)
    if family == "uneven":
        lo = _log_int(rng, 300, 3_000)
        return _run_case(None, kind, lo, _log_int(rng, 16, 256), min(steps, 2_000), points, f=f, period=period,
                         uneven_to=lo * rng.randint(4, 16), fp64=rng.random() < 0.3)
    # Sites in all: from a single short line up to what keeps the pass within the listed costs.
    fp64 = family == "fp64"
    most = min((1.2e10 if fp64 else 1.2e11) / steps, 2.0e7)
    sites = _log_int(rng, 200, max(most, 400))
    samples = min(_log_int(rng, 1, 64), max(1, sites // 100))
    return _run_case(None, kind, max(3, sites // samples + rng.randint(-3, 3)), samples, steps, points, f=f,
                     period=period, fp64=fp64, states=samples if sites < 50_000 else 1)


def _problem(case, seed):
    base = (int(seed) * 0x9E3779B97F4A7C15 + 0x1211_7275) & 0xFFFFFFFFFFFFFFFF
    n = case["samples"]
    if case["uneven_to"]:
        rng = np.random.Generator(np.random.PCG64(case["L"]))  # the sizes belong to the case
        lens = np.exp(rng.uniform(np.log(case["L"]), np.log(case["uneven_to"]), size=n))
        L = np.maximum(np.round(lens).astype(np.int64), 3)
    else:
        L = np.full(n, case["L"], np.int64)
    drives = case["f"] + case["spacing"] * np.arange(case["drives"])
    edges = None
    if case["sq_bins"] < 0:
        edges = workloads.sq_edges_full(case["L"])
    elif case["sq_bins"] > 0:
        edges = workloads.sq_edges_log(case["L"], case["sq_bins"])
    return workloads.custom(case["kind"], np.tile(L, case["drives"]), np.repeat(drives, n), case["steps"],
                            workloads.log_steps(case["steps"], case["points"]), base,
                            disorder_id=np.tile(np.arange(n), case["drives"]), c=C, dt=DT,
                            period=case["period"], sq_edges=edges)


def _seed63(seed):
    return (int(seed) * 0x2545F4914F6CDD1D + 0x5EED) & 0x7FFFFFFFFFFFFFFF


def prepare(case, seed):
    if case["call"] == "run":
        p = _problem(case, seed)
        if case["fp64"]:
            sim = qew.Simulation(p, precision=qew.QEW_FP64_PLAIN, path=qew.QEW_ONE_STEP)
        else:
            sim = qew.Simulation(p, k=case["k"], tile=case["tile"])
            if not (case["k"] and case["tile"]):
                sim.autotune()
        return {"case": case, "sim": sim}
    if case["call"] == "critical":
        return {"case": case, "seed": _seed63(seed), "ids": np.arange(case["samples"])}
    drives = np.geomspace(case["f_min"], case["f_max"], case["drives"])
    return {"case": case, "seed": _seed63(seed), "drives": drives}


def run(state):
    case = state["case"]
    if case["call"] == "run":
        sim = state["sim"]
        out = sim.run()
        out["ensemble"] = sim.ensemble()
        if case["sq_bins"]:
            out["sq"] = sim.structure_factor()
        if case["states"]:
            out["u"] = np.concatenate([sim.read_state(s)[0] for s in range(case["states"])])
        return out
    if case["call"] == "critical":
        return critical.critical_forces(case["kind"], case["L"], case["M"], state["ids"], state["seed"],
                                        f_hi=case["f_hi"], tol_f=case["tol_f"])
    r = std.fscan(case["kind"], case["L"], state["drives"], case["steps"], case["points"], state["seed"],
                  disorders=case["disorders"])
    return {k: r[k] for k in ("t", "drives", "v", "w2", "signs")}


def work(case):
    if case["call"] == "critical":
        # Every site passes each of its M cells once in each trial that depins (about half of the
        # halvings): a window of nodes, the local force and its zero, some 40 operations.
        rounds = math.ceil(math.log2(case["f_hi"] / case["tol_f"]))
        sites = case["samples"] * case["L"]
        return {"bytes": sites * 16 + case["samples"] * 32, "flops": 40.0 * sites * case["M"] * rounds / 2}
    if case["call"] == "fscan":
        samples, fp64, points = case["drives"] * case["disorders"], False, case["points"]
        sites, modes = samples * case["L"], 0
    else:
        samples, fp64, points = case["samples"] * case["drives"], case["fp64"], case["points"]
        if case["uneven_to"]:  # mean of the log-uniform lengths
            lo, hi = case["L"], case["uneven_to"]
            sites = samples * (hi - lo) / math.log(hi / lo)
        else:
            sites = samples * case["L"]
        modes = sites if case["sq_bins"] else 0
    # A site update: Laplacian 3, cubic 6, total force 3, Euler 2, cell and offset 2 operations.
    flops = 16.0 * sites * case["steps"]
    # The FFT of a measurement: 5/2 L log2 L operations for a real line.
    if modes:
        flops += points * 2.5 * modes * math.log2(case["L"])
    # The state written once, the series of v, w2 and ubar.
    return {"bytes": 8.0 * sites + 24.0 * samples * points, "flops": flops}


# ---------------------------------------------------------------------------
# The same results in plain FP64 torch.
# ---------------------------------------------------------------------------
_MASK = 0xFFFFFFFF


def _philox_words(j, n, did, seed):
    """First two words of Philox4x32-10 of the counters (j, n, did, 0)."""
    x0, x1, x2, x3 = j & _MASK, n & _MASK, did & _MASK, torch.zeros_like(j)
    k0, k1 = seed & _MASK, (seed >> 32) & _MASK
    for _ in range(10):
        p0, p1 = x0 * 0xD2511F53, x2 * 0xCD9E8D57  # modulo 2^64: the bits are the product's
        x0, x1, x2, x3 = ((p1 >> 32) & _MASK) ^ x1 ^ k0, p1 & _MASK, ((p0 >> 32) & _MASK) ^ x3 ^ k1, p0 & _MASK
        k0, k1 = (k0 + 0x9E3779B9) & _MASK, (k1 + 0xBB67AE85) & _MASK
    return x0, x1


def _node(kind, seed, period, did, j, n):
    if period > 0:
        n = torch.remainder(n, period)
    x0, x1 = _philox_words(j, n, did, seed)
    if kind == RF:
        return (2 * (x0 >> 8) + 1 - (1 << 24)).to(torch.float64) / 16777216.0
    u1 = (2 * (x0 >> 9) + 1).to(torch.float64) / 16777216.0
    u2 = (2 * (x1 >> 9) + 1).to(torch.float64) / 16777216.0
    return torch.sqrt(-2.0 * torch.log(u1)) * torch.cos(2.0 * math.pi * u2)


def _coefficients(kind, p):
    """Pinning force in the offset s of a cell with nodes p[0..3]: a0 + s (a1 + s (a2 + s a3))."""
    zero = torch.zeros_like(p[0])
    if kind == RB_LIN:
        return p[1] - p[2], zero, zero, zero
    if kind == RF_PC:
        return p[1], zero, zero, zero
    c1 = p[2] - p[0]
    c2 = 2.0 * p[0] - 5.0 * p[1] + 4.0 * p[2] - p[3]
    c3 = 3.0 * (p[1] - p[2]) + (p[3] - p[0])
    if kind == RF:
        return p[1], 0.5 * c1, 0.5 * c2, 0.5 * c3
    return -0.5 * c1, -c2, -1.5 * c3, zero


def _simulate(p):
    """Series v, w2, ubar [S][n_meas], the binned structure factor (or None) and the final states."""
    dev = torch.device("cuda")
    L = np.asarray(p["L"], np.int64)
    S, kind, seed, period = L.size, p["kind"], p["seed"], p["period"]
    off = np.concatenate([[0], np.cumsum(L)])
    lens = torch.from_numpy(L).to(dev)
    sample = torch.repeat_interleave(torch.arange(S, device=dev), lens)
    first = torch.from_numpy(off[:-1].copy()).to(dev)[sample]
    j = torch.arange(int(off[-1]), device=dev) - first
    equal = bool(np.all(L == L[0]))
    if not equal:
        left = first + torch.remainder(j - 1, lens[sample])
        right = first + torch.remainder(j + 1, lens[sample])
    del first
    did = torch.from_numpy(np.asarray(p["disorder_id"], np.int64)).to(dev)[sample]
    f = torch.from_numpy(np.asarray(p["f"], np.float64)).to(dev)[sample]
    u = torch.zeros(j.numel(), dtype=torch.float64, device=dev)
    cell = torch.zeros_like(j)
    a = torch.stack(_coefficients(kind, [_node(kind, seed, period, did, j, cell - 1 + i) for i in range(4)]))
    cell = cell.to(torch.float64)

    def force():
        if equal:
            g = u.view(S, -1)
            lap = (torch.roll(g, 1, 1) + torch.roll(g, -1, 1)).view(-1) - 2.0 * u
        else:
            lap = u[left] + u[right] - 2.0 * u
        s = u - cell
        return C * lap + f + (a[0] + s * (a[1] + s * (a[2] + s * a[3])))

    def mean(x):
        if equal:
            return x.view(S, -1).mean(1)
        return torch.stack([x[off[s]:off[s + 1]].mean() for s in range(S)])

    n_meas = len(p["meas_steps"])
    out = {k: np.full((S, n_meas), np.nan) for k in ("v", "w2", "ubar")}
    edges = p.get("sq_edges")
    sq = None if edges is None else np.zeros((n_meas, len(edges) - 1))
    at = {int(m): i for i, m in enumerate(p["meas_steps"])}
    for step in range(p["n_steps"] + 1):
        F = force()
        if step in at:
            i = at[step]
            ub = mean(u)
            out["v"][:, i] = mean(F).cpu().numpy()
            out["ubar"][:, i] = ub.cpu().numpy()
            out["w2"][:, i] = mean((u - ub[sample]) ** 2).cpu().numpy()
            if sq is not None:
                modes = (torch.fft.rfft(u.view(S, -1) - ub[:, None], dim=1).abs() / int(L[0])) ** 2
                line = modes.mean(0).cpu().numpy()
                for b in range(len(edges) - 1):
                    sq[i, b] = line[edges[b]:edges[b + 1]].mean()
                del modes
        if step == p["n_steps"]:
            break
        u = u + DT * F
        new = torch.floor(u)
        moved = torch.nonzero(new != cell).view(-1)
        if moved.numel():
            nm = new[moved].to(torch.int64)
            a[:, moved] = torch.stack(_coefficients(
                kind, [_node(kind, seed, period, did[moved], j[moved], nm - 1 + i) for i in range(4)]))
            cell = new
    return out, sq, u


def exact(case, seed):
    if case["call"] == "critical":
        return None  # the iteration needs too many sweeps for plain torch
    if case["call"] == "fscan":
        samples = case["drives"] * case["disorders"]
        sites, discontinuous = samples * case["L"], False
    else:
        samples, discontinuous = case["samples"] * case["drives"], case["kind"] in (RB_LIN, RF_PC)
        sites = samples * (case["uneven_to"] or case["L"])
    if case["steps"] * (1.2e-3 + sites * 4e-10) > 18.0:
        return None
    if discontinuous and not case.get("fp64", False):
        return None  # the force jumps at the integers: FP32 offsets take another branch there
    if case["call"] == "fscan":
        drives = np.geomspace(case["f_min"], case["f_max"], case["drives"])
        d = case["disorders"]
        p = workloads.custom(case["kind"], [case["L"]] * samples, np.repeat(drives, d), case["steps"],
                             workloads.log_steps(case["steps"], case["points"]), _seed63(seed),
                             disorder_id=np.tile(np.arange(d), drives.size), c=C, dt=DT)
        out, _, _ = _simulate(p)
        v = out["v"].reshape(drives.size, d, -1).mean(1)
        w2 = out["w2"].reshape(drives.size, d, -1).mean(1)
        return {"t": p["meas_steps"] * DT, "drives": drives, "v": v, "w2": w2, "signs": None}
    p = _problem(case, seed)
    out, sq, u = _simulate(p)
    S = len(p["L"])
    se = {k: (out[k].std(0, ddof=1) / math.sqrt(S) if S > 1 else np.zeros(out[k].shape[1])) for k in out}
    ens = {}
    for k in ("v", "w2", "ubar"):
        ens[k] = out[k].mean(0)
        ens[k + "_se"] = se[k]
    ens["w2_about_ensemble_ubar"] = out["w2"].mean(0) + out["ubar"].var(0)
    out["ensemble"] = ens
    if sq is not None:
        out["sq"] = sq
    if case["states"]:
        out["u"] = u[:int(np.sum(p["L"][:case["states"]]))].cpu().numpy()
    return out
