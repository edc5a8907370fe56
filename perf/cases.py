"""The work that a program has this library do, as cases that can be timed.

Every case is a dict of plain values with the field "kind":

  opacity    hk_opacity of a resident line list and, where "bin" > 0, hk_kdist
             of the grid: the step of a run over one atmosphere layer
  tables     hk_tables: k(g) over a table of (T, P) states
  stream     hk_opacity_stream: a list too long to hold, in pieces from host
             memory
  mixture    per species hk_load_lines (device arrays) and an accumulated
             hk_opacity, then hk_kdist: a mixed atmosphere layer
  fit        hk_kdist with the sorted bins kept, hk_resample and
             hk_transmission of an opacity grid at hand
  direct     hk_transmission_direct of sorted bins at hand
  train      hk_surrogate_set_params, hk_surrogate_train and the trained
             parameters: one stretch of fitting the Voigt surrogate

The line lists are drawn as the repository's synthetic ones are (uniform in
wavenumber and in log strength, exponential lower-state energies, uniform
widths and exponents), the column masses as in its benchmark.
"""
import math

import numpy as np
import torch

import paper_1503_03806_amd as hk

ATM_PER_BAR = 1.0 / 1.01325
T_REF = 296.0
N_G = 20
DEV = "cuda:0"


def listed():
    return [
        # one narrow band of a small molecule: what an interactive user or a
        # retrieval's inner loop asks for, where launches and latency count
        {"name": "band_500_f64", "kind": "opacity", "precision": "f64", "lines": 500, "nu0": 2000.0, "dnu": 0.01,
         "points": 6017, "cutoff": 5.0, "lorentz": 0.0, "T": 1500.0, "P": 1.0, "bin": 0, "rule": 0, "full": False},
        # a small molecule's whole list at the paper's resolution, bins of 1e5
        {"name": "list_1e4_f64", "kind": "opacity", "precision": "f64", "lines": 10000, "nu0": 0.0, "dnu": 0.01,
         "points": 300000, "cutoff": 25.0, "lorentz": 0.0, "T": 1500.0, "P": 1.0, "bin": 100000, "rule": 0,
         "full": False},
        # the benchmark's step: 1e6 lines, 3e6 points, 300 bins, binary64
        {"name": "list_1e6_f64", "kind": "opacity", "precision": "f64", "lines": 1000000, "nu0": 0.0, "dnu": 0.01,
         "points": 3000000, "cutoff": 100.0, "lorentz": 0.0, "T": 1500.0, "P": 1.0, "bin": 10000, "rule": 0,
         "full": False},
        # the same step with binary32 profiles
        {"name": "list_1e6_f32", "kind": "opacity", "precision": "f32", "lines": 1000000, "nu0": 0.0, "dnu": 0.01,
         "points": 3000000, "cutoff": 100.0, "lorentz": 0.0, "T": 1500.0, "P": 1.0, "bin": 10000, "rule": 0,
         "full": False},
        # a hot, dense list with every optional field, the cutoff in Lorentz
        # widths, ragged bins and the midpoint-linear rule
        {"name": "dense_3e6_f64", "kind": "opacity", "precision": "f64", "lines": 3000000, "nu0": 500.0, "dnu": 0.01,
         "points": 1000003, "cutoff": 0.0, "lorentz": 500.0, "T": 2000.0, "P": 0.8, "bin": 5000, "rule": 1,
         "full": True},
        # a k-distribution table in the library's default precision
        {"name": "tables_16_f32", "kind": "tables", "precision": "f32", "lines": 200000, "nu0": 0.0, "dnu": 0.01,
         "points": 1000000, "cutoff": 25.0, "states": 16, "bin": 10000, "rule": 0},
        # the same in binary64, ragged sizes
        {"name": "tables_9_f64", "kind": "tables", "precision": "f64", "lines": 100000, "nu0": 1000.0, "dnu": 0.01,
         "points": 400021, "cutoff": 25.0, "states": 9, "bin": 4999, "rule": 0},
        # a database in files: eight wavenumber-ordered pieces of one list
        {"name": "stream_8_f64", "kind": "stream", "precision": "f64", "lines": 1000000, "nu0": 0.0, "dnu": 0.01,
         "points": 1000000, "cutoff": 25.0, "pieces": 8, "T": 1500.0, "P": 0.1},
        # two species mixed before the k-distribution, their (unordered)
        # lists held in device memory
        {"name": "mixture_2_f64", "kind": "mixture", "precision": "f64", "lines": 300000, "species": 2, "nu0": 0.0,
         "dnu": 0.01, "points": 1000000, "cutoff": 25.0, "T": 1000.0, "P": 1.0, "bin": 10000},
        # the fit of ln kappa(y) and the transmission at 1000 column masses
        {"name": "fit_300_f64", "kind": "fit", "precision": "f64", "points": 2994321, "bin": 10000, "coef": 20,
         "columns": 1000},
        # the transmission of the same sort of bins without the fit
        {"name": "direct_100_f64", "kind": "direct", "precision": "f64", "points": 1000000, "bin": 10000,
         "columns": 500},
        # fitting the surrogate: 64 Adam steps of the recipe's batch
        {"name": "train_64", "kind": "train", "samples": 262144, "batch": 4096, "steps": 64, "lr": 1e-3,
         "wscale": 3.0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["opacity", "opacity", "opacity", "tables", "stream", "mixture", "fit", "direct", "train"])
    c = {"kind": kind}
    if kind == "train":
        c.update(samples=_log_int(rng, 5000, 500000), batch=_log_int(rng, 256, 8192), steps=rng.randint(4, 64),
                 lr=10.0 ** rng.uniform(-4.0, -2.5), wscale=rng.choice([0.0, 3.0]))
        return c
    c["precision"] = rng.choice(["f64", "f64", "f32"])
    if kind in ("fit", "direct"):
        c["points"] = _log_int(rng, 20000, 3000000 if kind == "fit" else 1000000)
        c["bin"] = min(_log_int(rng, 500, 50000), c["points"])
        if 0 < c["points"] % c["bin"] < 32:  # every bin holds at least as many points as coefficients
            c["points"] += 32
        c["columns"] = _log_int(rng, 10, 1000 if kind == "fit" else 500)
        if kind == "fit":
            c["coef"] = rng.randint(4, 32)
        return c
    c["points"] = _log_int(rng, 5000, 2000000)
    c["dnu"] = rng.choice([0.01, 0.01, 0.0078125, 0.02, 0.005])
    c["nu0"] = rng.choice([0.0, 500.0, 2000.0, 5000.0])
    span = c["points"] * c["dnu"]
    c["cutoff"] = math.exp(rng.uniform(math.log(2.0), math.log(100.0)))
    states = rng.randint(2, 12) if kind == "tables" else 1
    # lines per cm^-1 from sparse to dense, within the work of the largest listed case
    most = min(1000000, 1.5e10 * c["dnu"] / (2.0 * c["cutoff"]) / states)
    c["lines"] = max(100, min(_log_int(rng, 100, 1000000), int(most), int(400.0 * span)))
    if kind == "tables":
        c.update(states=states, bin=min(_log_int(rng, 500, 30000), c["points"]), rule=rng.randint(0, 1))
        return c
    c["T"] = math.exp(rng.uniform(math.log(300.0), math.log(3000.0)))
    c["P"] = 10.0 ** rng.uniform(-4.0, 1.0)
    if kind == "opacity":
        c.update(lorentz=rng.choice([0.0, 0.0, 0.0, 500.0]), full=rng.random() < 0.3, rule=rng.randint(0, 1),
                 bin=rng.choice([0, min(_log_int(rng, 500, 120000), c["points"])]))
        if c["lorentz"] > 0.0:
            c["P"] = 10.0 ** rng.uniform(-2.0, 0.0)
            c["T"] = math.exp(rng.uniform(math.log(1000.0), math.log(3000.0)))
    elif kind == "stream":
        c["pieces"] = rng.randint(1, 12)
    else:
        c.update(species=rng.randint(2, 3), bin=min(_log_int(rng, 500, 30000), c["points"]))
        c["lines"] = max(100, c["lines"] // c["species"])
    return c


# ---- inputs, from the seed alone ----------------------------------------------


def _line_list(n, lo, hi, seed, full=False):
    r = np.random.default_rng(seed)
    d = {"nu": np.maximum(r.uniform(lo, hi, n), 1e-6), "S_ref": 10.0 ** r.uniform(-30.0, -18.0, n),
         "E_lower": r.exponential(2000.0, n), "gamma_air": r.uniform(0.02, 0.1, n), "n_air": r.uniform(0.4, 0.8, n)}
    if full:
        d["gamma_self"] = r.uniform(0.1, 0.5, n)
        d["delta"] = r.uniform(-0.02, 0.02, n)
        d["A21"] = 10.0 ** r.uniform(0.0, 6.0, n)
    return d


def _sorted(d):
    o = np.argsort(d["nu"], kind="stable")
    return {k: np.ascontiguousarray(v[o]) for k, v in d.items()}


def _state(T, P, abundance=1.0):
    return {"T": T, "P": P, "P_self": 0.5 * P, "q_ratio": (T_REF / T) ** 1.5, "abundance": abundance}


def _table_states(c):
    """A table's corner-to-corner spread: T geometric, P geometric, paired cyclically."""
    n = c["states"]
    Ts = np.geomspace(300.0, 3000.0, n)
    Ps = np.geomspace(1e-6, 100.0, n) * ATM_PER_BAR
    return [_state(float(Ts[i]), float(Ps[(3 * i + 1) % n])) for i in range(n)]


def _grid(c):
    return {"nu_min": c["nu0"], "dnu": c["dnu"], "n_points": c["points"], "cutoff": c["cutoff"],
            "cutoff_lorentz": c.get("lorentz", 0.0)}


def _lists(c, seed):
    """The line lists of a case: one, or one per species."""
    hi = c["nu0"] + c["points"] * c["dnu"]
    k = c.get("species", 1)
    got = [_line_list(c["lines"], c["nu0"], hi, (int(seed), s), c.get("full", False)) for s in range(k)]
    return [_sorted(d) for d in got] if c["kind"] == "stream" else got


def _masses(c):
    return [18.0, 44.0, 16.0][:c.get("species", 1)]


def _abundances(c):
    return {1: [1.0], 2: [0.7, 0.3], 3: [0.6, 0.3, 0.1]}[c.get("species", 1)]


def _g_nodes():
    x, _ = np.polynomial.legendre.leggauss(N_G)
    return 0.5 * (1.0 + x)


def _columns(n):
    return torch.tensor(np.logspace(-18.0, 30.0, n), device=DEV)


def _kappa_grid(c, seed):
    """An opacity grid as a dense list gives it: per bin a base over eight
    decades, within it Lorentz-like peaks over several."""
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    n = c["points"]
    bins = -(-n // c["bin"])
    base = 10.0 ** (torch.rand(bins, generator=gen, device=DEV, dtype=torch.float64) * 8.0 - 28.0)
    u = torch.rand(n, generator=gen, device=DEV, dtype=torch.float64)
    k = base.repeat_interleave(c["bin"])[:n] / (u * u + 1e-5)
    if c["precision"] == "f32":
        k = (k * 1e22).to(torch.float32)  # in units that binary32 holds
    return k


def _train_inputs(c, seed):
    r = np.random.default_rng(int(seed))
    x = r.uniform(0.0, 50.0, c["samples"]).astype(np.float32)
    y = (10.0 ** r.uniform(-4.0, 2.0, c["samples"])).astype(np.float32)
    parts = []
    for shape, fan in (((64, 2), 2), ((64,), 0), ((64, 64), 64), ((64,), 0), ((64, 64), 64), ((64,), 0),
                       ((64, 64), 64), ((64,), 0), ((64,), 64), ((1,), 0)):
        n = int(np.prod(shape))
        parts.append(r.uniform(-1.0, 1.0, n) * math.sqrt(6.0 / fan) if fan else np.zeros(n))
    return x, y, np.concatenate(parts).astype(np.float32)


# ---- a program's state and one pass ---------------------------------------------


def _precision(c):
    return hk.HK_F64 if c["precision"] == "f64" else hk.HK_F32_KAHAN


def prepare(case, seed):
    c = case
    ctx = hk.Context(0)
    s = {"c": c, "ctx": ctx}
    kind = c["kind"]
    if kind == "train":
        x, y, s["theta"] = _train_inputs(c, seed)
        s["x"], s["y"] = torch.from_numpy(x).to(DEV), torch.from_numpy(y).to(DEV)
        s["z"] = ctx.surrogate_labels(s["x"], s["y"])
        return s
    s["prec"] = _precision(c)
    if kind in ("fit", "direct"):
        k = _kappa_grid(c, seed)
        s["m"] = _columns(c["columns"])
        s["g"] = _g_nodes()
        if kind == "direct":
            s["sorted"] = torch.empty_like(k)
            ctx.kdist(k, c["bin"], s["g"], s["prec"], sorted_out=s["sorted"])
        else:
            s["kappa"], s["sorted"] = k, torch.empty_like(k)
        return s
    s["grid"], s["g"] = _grid(c), _g_nodes()
    lists = _lists(c, seed)
    if kind == "tables":
        s["states"] = _table_states(c)
        ctx.load_lines(lists[0], 18.0, T_REF)
    elif kind == "stream":
        edges = np.linspace(0, c["lines"], c["pieces"] + 1).astype(np.int64)
        s["pieces"] = [{k: np.ascontiguousarray(v[a:b]) for k, v in lists[0].items()}
                       for a, b in zip(edges[:-1], edges[1:])]
        s["state"] = _state(c["T"], c["P"])
    elif kind == "mixture":
        s["lists"] = [{k: torch.from_numpy(v).to(DEV) for k, v in d.items()} for d in lists]
        s["kappa"] = torch.empty(c["points"], dtype=torch.float64, device=DEV)
    else:
        s["state"] = _state(c["T"], c["P"])
        ctx.load_lines(lists[0], 18.0, T_REF)
    return s


def run(state):
    s = state
    c, ctx, kind = s["c"], s["ctx"], s["c"]["kind"]
    if kind == "opacity":
        kappa = ctx.opacity(s["state"], s["grid"], s["prec"])
        if not c["bin"]:
            return {"kappa": kappa}
        return {"kappa": kappa, "k": ctx.kdist(kappa, c["bin"], s["g"], rule=c["rule"])}
    if kind == "tables":
        return {"k": ctx.tables(s["states"], s["grid"], c["bin"], s["g"], s["prec"], rule=c["rule"])}
    if kind == "stream":
        return {"kappa": ctx.opacity_stream(s["pieces"], 18.0, s["state"], s["grid"], s["prec"], T_ref=T_REF)}
    if kind == "mixture":
        kappa = s["kappa"]
        for i, (lines, mass, x) in enumerate(zip(s["lists"], _masses(c), _abundances(c))):
            ctx.load_lines(lines, mass, T_REF)
            ctx.opacity(_state(c["T"], c["P"], x), s["grid"], s["prec"], out=kappa, accumulate=i > 0)
        return {"kappa": kappa, "k": ctx.kdist(kappa, c["bin"], s["g"])}
    if kind == "fit":
        k = ctx.kdist(s["kappa"], c["bin"], s["g"], s["prec"], sorted_out=s["sorted"])
        coef = ctx.resample(s["sorted"], c["bin"], c["coef"], s["prec"])
        return {"k": k, "sorted": s["sorted"], "coef": coef, "T": ctx.transmission(coef, s["m"])}
    if kind == "direct":
        return {"T": ctx.transmission_direct(s["sorted"], c["bin"], s["m"], s["prec"])}
    ctx.surrogate_set_params(s["theta"])
    loss = ctx.surrogate_train(s["x"], s["y"], s["z"], c["batch"], c["steps"], c["lr"], wscale=c["wscale"])
    return {"loss": loss, "theta": ctx.surrogate_params()}


# ---- what a pass cannot do without ------------------------------------------------


def _mean_window(c, P, T):
    """Mean points of a line's window on the grid."""
    cut = c["cutoff"]
    if c.get("lorentz", 0.0) > 0.0:
        width = 0.18 if c.get("full", False) else 0.06
        cut = c["lorentz"] * width * P * (T / T_REF) ** -0.6
    return min(2.0 * cut / c["dnu"], float(c["points"]))


def _sort_flops(n, m):
    return n * max(1.0, math.log2(max(m, 2)))


def work(case):
    """Bytes: inputs read once, outputs written once.  Operations: of the
    profile scheme as the method states it, about 12 per line-point evaluation
    (Gauss-Hermite rules), comparisons of the sort, and so on."""
    c = case
    kind = c["kind"]
    if kind == "train":
        per = 2.0 * 3.0 * (2 * 64 + 3 * 64 * 64 + 64)  # forward, and the two products of the backward
        n = float(c["batch"]) * c["steps"]
        return {"bytes": 12.0 * n + 12737 * 4.0 * 2, "flops": per * n}
    n = float(c["points"])
    key = 8.0 if c["precision"] == "f64" else 4.0
    if kind in ("fit", "direct"):
        bins = -(-c["points"] // c["bin"])
        if kind == "direct":
            return {"bytes": n * key + 8.0 * c["columns"] * (1 + bins), "flops": 20.0 * n * c["columns"]}
        return {"bytes": 2 * n * key + 8.0 * bins * (N_G + c["coef"] + c["columns"]),
                "flops": _sort_flops(n, c["bin"]) + n * (20.0 + 2.0 * c["coef"]) + 20.0 * bins * 100 * c["columns"]}
    lines = float(c["lines"]) * c.get("species", 1)
    fields = 8 if c.get("full", False) else 5
    if kind == "tables":
        per = sum(lines * _mean_window(c, st["P"], st["T"]) for st in _table_states(c))
        bins = -(-c["points"] // c["bin"])
        return {"bytes": lines * 8.0 * fields + 8.0 * bins * N_G * c["states"],
                "flops": 12.0 * per + c["states"] * _sort_flops(n, c["bin"])}
    evals = lines * _mean_window(c, c["P"], c["T"])
    out = 8.0 * n
    flops = 12.0 * evals
    if c.get("bin", 0):
        out += 8.0 * -(-c["points"] // c["bin"]) * N_G
        flops += _sort_flops(n, c["bin"])
    return {"bytes": lines * 8.0 * fields + out, "flops": flops}


# ---- the same results in 64 bits, without the library -------------------------------

_C, _KB, _H, _AMU = 2.99792458e10, 1.380649e-16, 6.62607015e-27, 1.66053906660e-24
_C2 = _H * _C / _KB


def _grid_points(c):
    """nu_j = nu_min + j dnu, rounded once."""
    j = np.arange(c["points"], dtype=np.longdouble)
    nu = j * np.longdouble(c["dnu"]) + np.longdouble(c["nu0"])
    return torch.from_numpy(nu.astype(np.float64)).to(DEV)


def _exact_kappa(c, lines, mass, st, nuj):
    """kappa(nu_j): S Phi summed over the lines whose window holds the point;
    the series form of the Faddeeva function for a^2 + u^2 < 100, the 3-node
    Gauss-Hermite rule below 1e6 and the 1-node rule beyond."""
    d = {k: torch.from_numpy(v).to(DEV) for k, v in _sorted(lines).items()}
    nu, T, P, Ps = d["nu"], st["T"], st["P"], st["P_self"]
    S = d["S_ref"] * (st["q_ratio"] * st["abundance"]) * torch.exp(-_C2 * d["E_lower"] / T + _C2 * d["E_lower"] / T_REF)
    S = S * (torch.expm1(-_C2 * nu / T) / torch.expm1(-_C2 * nu / T_REF))
    al = nu * (math.sqrt(2.0 * _KB * T / (mass * _AMU)) / _C)
    G = (T / T_REF) ** (-d["n_air"]) * (d["gamma_air"] * (P - Ps) + d.get("gamma_self", d["gamma_air"]) * Ps)
    if "A21" in d:
        G = G + d["A21"] / (4.0 * math.pi * _C)
    nu0 = nu + d["delta"] * P if "delta" in d else nu
    n, dnu, nmin = c["points"], c["dnu"], c["nu0"]
    cut = c["lorentz"] * G if c.get("lorentz", 0.0) > 0.0 else torch.full_like(nu, c["cutoff"])
    wlo = torch.ceil((nu0 - cut - nmin) / dnu)
    whi = torch.floor((nu0 + cut - nmin) / dnu)
    a = G / al
    a2, inva, G2, Lg = a * a, 1.0 / al, G * G, S * G / math.pi
    s3, norm, ecx = math.sqrt(1.5) * al, S / (al * math.sqrt(math.pi)), torch.special.erfcx(a)
    reach = float(cut.max()) + (float((nu0 - nu).abs().max()) if len(nu) else 0.0) + 2.0 * dnu
    out = torch.zeros(n, dtype=torch.float64, device=DEV)
    hn = 0.5 * torch.arange(1, 41, dtype=torch.float64, device=DEV)
    wide = max(64, min(4096, int(2.5e7 / max(1.0, float(len(nu)) * min(1.0, 2.0 * reach / (n * dnu))))))
    first = torch.searchsorted(nu, nuj[::wide] - reach).tolist()
    ends = torch.arange(wide - 1, n + wide - 1, wide, device=DEV)
    last = torch.searchsorted(nu, nuj[torch.clamp(ends, max=n - 1)] + reach, right=True).tolist()
    for b, (l0, l1) in enumerate(zip(first, last)):
        j0, j1 = b * wide, min((b + 1) * wide, n)
        for k0 in range(l0, l1, 50000):  # a dense list, some lines at a time
            k = slice(k0, min(l1, k0 + 50000))
            jj = torch.arange(j0, j1, dtype=torch.float64, device=DEV)[:, None]
            dv = nuj[j0:j1, None] - nu0[k]
            u = dv.abs() * inva[k]
            r2 = u * u + a2[k]
            one = 1.0 / (dv * dv + G2[k])
            three = one * (2.0 / 3.0) + (1.0 / ((dv - s3[k]) ** 2 + G2[k]) + 1.0 / ((dv + s3[k]) ** 2 + G2[k])) / 6.0
            inside = (jj >= wlo[k]) & (jj <= whi[k])
            core = inside & (r2 < 100.0)
            v = torch.where(r2 >= 1.0e6, one, three) * Lg[k]
            out[j0:j1] += torch.where(inside & ~core, v, 0.0).sum(1)
            p, q = core.nonzero(as_tuple=True)
            for i in range(0, len(p), 400000):
                pi, qi = p[i:i + 400000], q[i:i + 400000]
                x, li = u[pi, qi], qi + k0
                y = a[li]
                w = 1.0 / (hn * hn + a2[li][:, None])
                E = torch.exp(-x * x)
                xe = x[:, None]
                s23 = ((torch.exp(-(hn - xe) ** 2) + torch.exp(-(hn + xe) ** 2)) * w).sum(1)
                t1 = (torch.exp(-hn * hn) * w).sum(1)
                c2, s = torch.cos(2.0 * x * y), torch.sin(x * y)
                H = E * (ecx[li] * c2 + s * s / (math.pi * y)) + (y / math.pi) * (0.5 * s23 - c2 * E * t1)
                out.index_add_(0, pi + j0, norm[li] * H)
    return out


def _k_of_g(srt, g, rule):
    m = len(srt)
    v = srt.to(torch.float64)
    got = []
    for gi in g:
        if rule == 0:
            got.append(v[min(max(math.ceil(gi * m) - 1, 0), m - 1)])
            continue
        u = gi * m - 0.5
        i = math.floor(u)
        got.append(v[0] if u <= 0 else v[m - 1] if i >= m - 1 else v[i] + (u - i) * (v[i + 1] - v[i]))
    return torch.stack(got)


def _exact_sort(kappa, size, g, rule):
    srt = torch.cat([torch.sort(kappa[i:i + size]).values for i in range(0, len(kappa), size)])
    return srt, torch.stack([_k_of_g(srt[i:i + size], g, rule) for i in range(0, len(kappa), size)])


def _exact_fit(srt, size, nc):
    coef = []
    for m, part in ((size, srt[:len(srt) // size * size].reshape(-1, size)),
                    (len(srt) % size, srt[len(srt) // size * size:].reshape(1, -1))):
        if part.numel() == 0:
            continue
        t = 2.0 * (torch.arange(m, dtype=torch.float64, device=DEV) + 0.5) / m - 1.0
        A = torch.stack([torch.cos(i * torch.acos(t)) for i in range(nc)], 1)
        Q, R = torch.linalg.qr(A)
        y = torch.log(part.to(torch.float64).clamp_min(2.2250738585072014e-308)) @ Q
        coef.append(torch.linalg.solve_triangular(R, y.T, upper=True).T)
    return torch.cat(coef)


def exact(case, seed):
    c = case
    kind = c["kind"]
    if kind == "train":
        return None  # a bfloat16 network's steps have no value in 64 bits
    if kind in ("fit", "direct"):
        kappa, m, g = _kappa_grid(c, seed), _columns(c["columns"]), _g_nodes()
        srt, k = _exact_sort(kappa, c["bin"], g, 0)
        if kind == "direct":
            T = []
            for i in range(0, len(srt), c["bin"]):
                v = srt[i:i + c["bin"]].to(torch.float64)
                T.append(torch.cat([torch.exp(-v[:, None] * mm).mean(0) for mm in m.split(64)]))
            return {"T": torch.stack(T)}
        coef = _exact_fit(srt, c["bin"], c["coef"])
        x, w = np.polynomial.legendre.leggauss(100)
        t = torch.from_numpy(x).to(DEV)
        B = torch.stack([torch.cos(i * torch.acos(t)) for i in range(c["coef"])])
        kq = torch.exp(coef @ B)
        wq = torch.from_numpy(0.5 * w).to(DEV)
        T = torch.stack([torch.exp(-kb[None, :] * m[:, None]) @ wq for kb in kq])
        return {"k": k, "sorted": srt, "coef": coef, "T": T}
    # about 4e9 evaluations take a second
    states = _table_states(c) if kind == "tables" else [_state(c["T"], c["P"])]
    pairs = sum(c["lines"] * c.get("species", 1) * _mean_window(c, st["P"], st["T"]) for st in states)
    if pairs > 4e10:
        return None
    nuj, g = _grid_points(c), _g_nodes()
    lists = _lists(c, seed)
    if kind == "tables":
        return {"k": torch.stack([_exact_sort(_exact_kappa(c, lists[0], 18.0, st, nuj), c["bin"], g, c["rule"])[1]
                                  for st in states])}
    kappa = torch.zeros_like(nuj)
    for lines, mass, x in zip(lists, _masses(c), _abundances(c)):
        kappa = kappa + _exact_kappa(c, lines, mass, _state(c["T"], c["P"], x), nuj)
    if not c.get("bin", 0):
        return {"kappa": kappa}
    return {"kappa": kappa, "k": _exact_sort(kappa, c["bin"], g, c.get("rule", 0))[1]}
