"""Performance cases: swarm runs as a program of this library makes them.

A case is a dict of plain values: the gas, the field, the precision, the options and the
sizes of the runs, and how the program calls the library:

  single  one handle, `run` and its tallies (and the per-electron records, where a program
          analyses them itself, as the FP32 bias study of bench.py does);
  batch   many handles in one batched launch: a scan of the reduced field (`scan`), or
          uneven runs of several mixtures (`uneven`);
  real    one handle whose ionisations create electrons;
  server  a server that takes a burst of requests with random gases and is drained.

Units: E/N in townsend, energies in eV, B in tesla.
"""
import math
from dataclasses import replace

import numpy as np
import torch

import paper_1901_08140_amd as sw
import synth

F32, F64 = "fp32", "fp64"
PRECISION = {F32: sw.SWARM_FP32_MIXED, F64: sw.SWARM_FP64}
DEFAULTS = {"gas": "argon", "td": 100.0, "b": 0.0, "angle": 0.0, "precision": F32, "option": "plain", "records": False,
            "instances": 1, "spread": "one"}


def _case(**kw):
    return {**DEFAULTS, **kw}


def listed():
    return [
        # A quick check of a new gas or field: a few waves of electrons for a moment, where
        # the call's own latency counts.
        _case(name="check_f32", kind="single", electrons=256, collisions=100),
        # The worked example of the paper (25 particles, Ar:CO2 93:7 at 2.4 Td), a tenth of its
        # 200000 interactions: very few electrons that run for long.
        _case(name="example_f64", kind="single", gas="arco2_93", td=2.4, precision=F64, electrons=25, collisions=20_000,
              records=True),
        # The Maxwell gas in full: the closed-form check of the method.
        _case(name="maxwell_f64", kind="single", gas="maxwell", td=10.0, precision=F64, electrons=1000, collisions=10_000,
              records=True),
        # One field point of the argon study in double precision, with the records.
        _case(name="point_f64", kind="single", precision=F64, electrons=100_000, collisions=2000, records=True),
        # One field point in mixed precision at the study's full size.
        _case(name="point_f32", kind="single", td=10.0, electrons=100_000, collisions=20_000),
        # A mid-sized magnetised mixture point (28 channels), odd sizes, moving targets.
        _case(name="warm_f32", kind="single", gas="arco2", td=31.0, b=1.0, angle=0.7, option="thermal", electrons=9_973,
              collisions=1_777),
        # The argon study: 32 fields from 1 to 1000 Td in one batched launch.
        _case(name="scan_f32", kind="batch", spread="scan", instances=32, electrons=100_000, collisions=20_000),
        # The same study in double precision with a tenth of the budget.
        _case(name="scan_f64", kind="batch", spread="scan", instances=32, precision=F64, electrons=100_000, collisions=2000),
        # The study with the paper's variable trial frequency.
        _case(name="scan_variable_f32", kind="batch", spread="scan", instances=16, option="variable", electrons=50_000,
              collisions=5000),
        # Uneven runs of four mixtures with and without a magnetic field.
        _case(name="uneven_f32", kind="batch", spread="uneven", instances=64, electrons=100_000, collisions=10_000),
        # An avalanche in the magnetised mixture: ionisations create electrons.
        _case(name="avalanche_f32", kind="real", gas="arco2", b=1.0, angle=math.pi / 4, electrons=100_000, collisions=2000),
        # A burst of requests with random gases to a server.
        _case(name="burst_f32", kind="server", instances=24, electrons=20_000, collisions=4000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["single", "single", "single", "batch", "real", "server"])
    precision = rng.choice([F32, F64])
    magnetic = rng.random() < 0.4
    c = _case(kind=kind, precision=precision, td=round(math.exp(rng.uniform(0.0, math.log(1000.0))), 3),
              b=round(rng.uniform(0.1, 2.0), 3) if magnetic else 0.0,
              angle=round(rng.uniform(0.0, math.pi), 3) if magnetic else 0.0)
    most = 1.0e9 if precision == F32 else 2.5e8       # collisions of all electrons
    if kind == "single":
        c["gas"] = rng.choice(["argon", "argon", "arco2", "arco2_93", "maxwell"])
        c["option"] = rng.choice(["plain", "plain", "plain", "variable", "binned", "thermal", "screened"])
        c["records"] = rng.random() < 0.5
        c["electrons"] = _log_int(rng, 25, 300_000)
        c["collisions"] = max(50, min(_log_int(rng, 100, 20_000), int(most / c["electrons"])))
    elif kind == "batch":
        c["spread"] = rng.choice(["scan", "uneven"])
        c["instances"] = _log_int(rng, 3, 48)
        c["option"] = rng.choice(["plain", "plain", "variable", "binned"]) if c["spread"] == "scan" else "plain"
        c["electrons"] = _log_int(rng, 1000, 100_000)
        c["collisions"] = max(200, min(_log_int(rng, 500, 10_000), int(4 * most / (c["electrons"] * c["instances"]))))
    elif kind == "real":
        c["gas"] = "arco2"
        c["td"] = round(math.exp(rng.uniform(math.log(30.0), math.log(100.0))), 3)
        c["electrons"] = _log_int(rng, 500, 60_000)
        c["collisions"] = _log_int(rng, 200, 1500)
    else:
        c["precision"] = F32
        c["td"], c["b"], c["angle"] = 100.0, 0.0, 0.0
        c["instances"] = _log_int(rng, 3, 24)
        c["electrons"] = _log_int(rng, 1500, 20_000)
        c["collisions"] = _log_int(rng, 300, 4000)
    return c


# ---- inputs -------------------------------------------------------------------------------
def _gas(name):
    if name == "maxwell":
        return [synth.maxwell_component(4.0)]
    if name == "arco2":
        return synth.mixture_ar_co2()
    if name == "arco2_93":
        return synth.mixture_ar_co2(0.93, 0.07)
    return [synth.argon_like()]


OPTIONS = {"plain": {}, "variable": {"trial_strategy": 1}, "binned": {"trial_strategy": 2},
           "thermal": {"thermal_targets": 1}, "screened": {}}


def _config(case, td=None):
    comps = _gas(case["gas"])
    if case["option"] == "screened":
        comps = [c.with_scattering(1) for c in comps]
    return synth.SwarmConfig(comps, synth.td_to_field(case["td"] if td is None else td), B_T=case["b"],
                             B_angle_rad=case["angle"], secondaries=synth.REAL if case["kind"] == "real" else synth.DUMMY,
                             **OPTIONS[case["option"]])


def _runs(case, seed):
    """(configuration, electrons, collisions) of every run of a batch or a burst."""
    n, ne, nc = case["instances"], case["electrons"], case["collisions"]
    if case["kind"] == "server":
        out = []
        for i in range(n):
            rng = np.random.default_rng([17, i])
            cfg = synth.cfg5_request(i)
            out.append((cfg, int(round(ne * 10 ** rng.uniform(-1.0, 0.0))), int(round(nc * 10 ** rng.uniform(-1.0, 0.0)))))
        return out
    tds = np.geomspace(1.0, 1000.0, n)
    if case["spread"] == "scan":
        return [(_config(case, float(td)), ne, nc) for td in tds]
    rng = np.random.default_rng(4)
    mixes = synth.cfg4_mixtures()
    out = []
    for i, td in enumerate(tds):
        b, angle = (1.0, rng.uniform(0.0, math.pi)) if rng.uniform() < 0.5 else (0.0, 0.0)
        cfg = synth.SwarmConfig(mixes[i % 4], synth.td_to_field(float(td)), B_T=b, B_angle_rad=angle)
        out.append((cfg, int(round(ne * 10 ** rng.uniform(-2.0, 0.0))), int(round(nc * 10 ** rng.uniform(-1.0, 0.0)))))
    return out


def prepare(case, seed):
    """The handles (tables built) or the server that a program keeps, and the seeds of its runs."""
    precision = PRECISION[case["precision"]]
    st = {"case": case, "seed": int(seed)}
    if case["kind"] in ("single", "real"):
        st["swarm"] = sw.Swarm.from_config(_config(case), precision)
    elif case["kind"] == "batch":
        runs = _runs(case, seed)
        st["swarms"] = [sw.Swarm.from_config(cfg, precision) for cfg, _, _ in runs]
        jobs = [(ne, nc, st["seed"] + 1000 * i) for i, (_, ne, nc) in enumerate(runs)]
        st["batch"] = _Batch(st["swarms"], jobs)
    else:
        st["runs"] = [(cfg.components, sw.params_from_config(replace(cfg), precision), ne, nc, st["seed"] + 1000 * i)
                      for i, (cfg, ne, nc) in enumerate(_runs(case, seed))]
        st["server"] = _Server(precision)
    return st


class _Batch:
    """Owns a batch handle (released with the state that holds it)."""

    def __init__(self, swarms, jobs):
        self.swarms = swarms
        self.h = sw.swarm_batch_create([s.h for s in swarms], jobs, {"use_graph": 1})

    def __del__(self, destroy=sw.swarm_batch_destroy):
        destroy(self.h)


class _Server:
    def __init__(self, precision):
        self.h = sw.swarm_server_create(16 << 30, precision, schedule=sw.SWARM_SCHEDULE_SHORTEST_FIRST)

    def __del__(self, destroy=sw.swarm_server_destroy):
        destroy(self.h)


# ---- one pass -----------------------------------------------------------------------------
STATS = {"drift": ["W", "Wx", "Wy", "Wz"], "energy": ["mean_energy", "mean_energy_after"],
         "diffusion": ["D", "DL", "DT", "D_vec", "DL_vec", "DT_vec"],
         "magnitude": ["sigma", "sigmaL", "sigmaT", "sigma_vec", "sigmaL_vec", "sigmaT_vec"],
         "townsend": ["alpha", "eta"]}
RATES = ["alpha_rate", "eta_rate"]
COUNTS = ["n_real", "n_null", "n_forbidden", "n_fail", "n_over", "n_electrons", "n_finished", "n_attached", "n_stuck",
          "n_created", "n_ionizations", "n_attachments", "n_dropped", "n_retry_failed"]


def _tallies(ts):
    out = {k: np.array([[t[n] for n in names] for t in ts], dtype=np.float64) for k, names in STATS.items()}
    out["rates"] = np.array([[t[n] for n in RATES] for t in ts], dtype=np.float64)
    out["efficiency"] = np.array([t["efficiency"] for t in ts], dtype=np.float64)
    out["majorant"] = np.array([t["majorant"] for t in ts], dtype=np.float64)
    out["counts"] = np.array([[t[n] for n in COUNTS] for t in ts], dtype=np.int64)
    return out


INTS = ["id", "flags", "k_start", "k_end", "G", "D", "n_forbidden", "n_over", "n_fail", "n_null", "blocks"]
REALS = ["r", "t", "sum_eps", "sum_epsp"]


def _records(rec):
    out = {"rec_" + n: np.ascontiguousarray(rec[n]) for n in REALS}
    out["rec_ints"] = np.stack([rec[n].astype(np.int64) for n in INTS])
    return out


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind in ("single", "real"):
        s = st["swarm"]
        s.run(case["electrons"], case["collisions"], st["seed"])
        out = _tallies([s.tallies()])
        if case["records"]:
            out.update(_records(s.records()))
        return out
    if kind == "batch":
        b = st["batch"].h
        sw.swarm_batch_launch(b)
        sw.swarm_batch_wait(b)
        return _tallies([sw.swarm_batch_tallies(b, i) for i in range(case["instances"])])
    srv = st["server"].h
    tickets = [sw.swarm_server_submit(srv, *r) for r in st["runs"]]
    sw.swarm_server_drain(srv)
    return _tallies([sw.swarm_server_poll(srv, t)[1] for t in tickets])


# ---- the least work -------------------------------------------------------------------------
# Trials per real collision (1/efficiency of the null-collision test) at 1, 3, 10, ... 1000 Td,
# and the lane operations of the method per trial and per real collision: random numbers,
# flight time, energy, rate lookup and test; channel, direction, energy transfer and sums.
TRIALS = {"maxwell": [1.0] * 7, "argon": [25.3, 11.8, 5.7, 4.0, 3.3, 2.7, 1.9],
          "arco2": [70.0, 23.8, 7.1, 4.3, 3.4, 2.7, 1.9], "arco2_93": [62.6, 20.1, 6.7, 4.2, 3.4, 2.7, 1.9]}
OPS = {F32: (38.0, 113.0), F64: (82.0, 184.0)}


def _trials(gas, td):
    return math.exp(float(np.interp(math.log10(td), [0.0, 0.477, 1.0, 1.477, 2.0, 2.477, 3.0], np.log(TRIALS[gas]))))


def work(case):
    if case["kind"] in ("batch", "server"):
        runs = [(ne, nc) for _, ne, nc in _runs(case, 0)]
    else:
        runs = [(case["electrons"], case["collisions"])]
    real = float(sum(ne * nc for ne, nc in runs))
    electrons = float(sum(ne for ne, _ in runs))
    if case["kind"] == "server":
        trials = 16.7
    elif case["kind"] == "batch":
        trials = 9.7 if case["spread"] == "uneven" else 4.1
    else:
        trials = _trials(case["gas"], case["td"])
    if case["option"] in ("variable", "binned"):
        trials = min(trials, 1.9)
    per_trial, per_real = OPS[case["precision"]]
    size = 4 if case["precision"] == F32 else 8
    table = len(runs) * 1665 * 2 * size
    return {"bytes": electrons * 104.0 + table, "flops": real * (trials * per_trial + per_real)}


# ---- the same in 64 bits --------------------------------------------------------------------
# A plain torch float64 run of the method, all electrons in step (each draws one block of two
# trials per step until it has made its collisions).  Only the FP64 plain single runs have such
# a value: an FP32 run leaves the FP64 history of an electron for good at its first null test
# that its rounding turns over, and what it then computes is another sample.  Runs whose steps
# would take too long give None.
QE, ME, AMU = 1.602176634e-19, 9.1093837015e-31, 1.66053906660e-27
P, EMIN, EMAX = 64, -14, 12
G = (EMAX - EMIN) * P + 1
MASK = 0xFFFFFFFF


def _philox(c0, c1, c2, c3, seed):
    k0, k1 = seed & MASK, (seed >> 32) & MASK
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = ((p1 >> 32) & MASK) ^ c1 ^ k0, p1 & MASK, ((p0 >> 32) & MASK) ^ c3 ^ k1, p0 & MASK
        k0, k1 = (k0 + 0x9E3779B9) & MASK, (k1 + 0xBB67AE85) & MASK
    return c0, c1, c2, c3


def _uniforms(block, tag, ids, seed):
    """The four 53-bit uniforms of a block from its two streams (tag and tag + 1)."""
    z = torch.zeros_like(block + ids)
    hi = _philox(z + block, z + tag, z + ids, z, seed)
    lo = _philox(z + block, z + tag + 1, z + ids, z, seed)
    return [h.double() * 2.0 ** -32 + (x >> 11).double() * 2.0 ** -53 for h, x in zip(hi, lo)]


def _sigma(ch, eps):
    """Cross-section with the extension rules: constant to the left for elastic channels, zero
    below the threshold and a ramp from it otherwise, the power law of the last two points to the right."""
    e, s, thr = ch.energy_eV, ch.sigma_m2, float(ch.threshold_eV)
    lead = ch.kind != synth.ELASTIC and e[0] > thr
    ee, ss = (np.concatenate([[thr], e]), np.concatenate([[0.0], s])) if lead else (e, s)
    out = np.interp(eps, ee, ss)
    right = eps > e[-1]
    if s[-2] > 0.0 and s[-1] > 0.0:
        k = math.log(s[-1] / s[-2]) / math.log(e[-1] / e[-2])
        out[right] = s[-1] * (eps[right] / e[-1]) ** k
    else:
        out[right] = 0.0
    if ch.kind != synth.ELASTIC:
        out[eps < thr] = 0.0
    return out


def _simulate(cfg, n, budget, seed, dev):
    f64 = dict(dtype=torch.float64, device=dev)
    nodes = np.array([math.ldexp(1.0 + (g % P) / P, EMIN + g // P) for g in range(G)])
    chans = [(c, ch) for c in cfg.components for ch in c.channels]
    rate = np.cumsum([c.fraction * cfg.N_per_m3 * _sigma(ch, nodes) * np.sqrt(2.0 * nodes * QE / ME) for c, ch in chans], axis=0)
    cum = torch.tensor(rate.T.copy(), **f64)                                  # G x channels
    step = torch.cat([cum[1:] - cum[:-1], torch.zeros_like(cum[:1])])
    nup = (1.0 + 2.0 ** -20) * float(cum[:, -1].max())
    col = lambda f: torch.tensor([float(f(c, ch)) for c, ch in chans], **f64)  # noqa: E731
    kind = torch.tensor([ch.kind for _, ch in chans], device=dev)
    mass = col(lambda c, ch: c.mass_amu * AMU)
    thr = col(lambda c, ch: ch.threshold_eV)
    onset = thr * ((ME + mass) / mass)
    c_ela, c_m = 2.0 * ME * mass / (ME + mass) ** 2, mass / (ME + mass)
    c_eps, c_speed = 0.5 * ME / QE, math.sqrt(2.0 * QE / ME)
    az, w = -QE * cfg.E_V_per_m / ME, QE * cfg.B_T / ME
    b = torch.tensor([math.sin(cfg.B_angle_rad), 0.0, math.cos(cfg.B_angle_rad)], **f64)
    ids = torch.arange(n, dtype=torch.int64, device=dev)

    def direction(uc, up):
        ct = 1.0 - 2.0 * uc
        s = torch.sqrt((1.0 - ct) * (1.0 + ct))
        return torch.stack([s * torch.cos(2.0 * math.pi * up), s * torch.sin(2.0 * math.pi * up), ct], 1)

    def flight(v, t):
        """Velocity and displacement after the time t in the uniform fields."""
        t = t[:, None]
        a = torch.zeros_like(v)
        a[:, 2] = az
        if cfg.B_T == 0.0:
            return v + a * t, v * t + a * (0.5 * t * t)
        drift = torch.zeros_like(v)
        drift[:, 1] = cfg.E_V_per_m * b[0] / cfg.B_T
        par, apar = (v @ b)[:, None] * b, az * b[2] * b
        u = v - par - drift
        x = torch.linalg.cross(b.expand_as(u), u)
        s, c, h = torch.sin(w * t), torch.cos(w * t), torch.sin(0.5 * w * t)
        return (par + apar * t + drift + u * c + x * s,
                (par + drift) * t + apar * (0.5 * t * t) + (u * s + x * (2.0 * h * h)) / w)

    def grid(eps):
        m, e = torch.frexp(eps)
        x = (2.0 * m - 1.0) * P
        g = (e.long() - 1 - EMIN) * P + torch.floor(x).long()
        wt = x - torch.floor(x)
        low, high = g < 0, g >= G - 1
        return torch.clamp(g, 0, G - 1), torch.where(low | high, torch.zeros_like(wt), wt), g >= G - 1

    u0 = _uniforms(torch.zeros_like(ids), 4, ids, seed)
    v = c_speed * math.sqrt(cfg.init_energy_eV) * direction(u0[0], u0[1])
    r = torch.zeros_like(v)
    zero = torch.zeros(n, **f64)
    t, flown, se, sep, gi, da = (zero.clone() for _ in range(6))
    k = torch.zeros_like(ids)
    for s in range(40 * budget + 1000):
        if s % 64 == 0:
            if bool((k >= budget).all()):
                break
            words = _uniforms(torch.arange(s, s + 64, device=dev)[:, None], 0, ids[None, :], seed)
        live = k < budget
        hit = torch.zeros_like(live)
        for j in (0, 1):
            trying = live & ~hit
            flown = torch.where(trying, flown - torch.log1p(-words[2 * j][s % 64]) / nup, flown)
            vf, dr = flight(v, flown)
            eps = c_eps * (vf * vf).sum(1)
            g, wt, over = grid(eps)
            x = words[2 * j + 1][s % 64] * nup
            real = trying & (x < cum[g, -1] + wt * step[g, -1])
            if j == 0:
                keep = (vf, dr, eps, g, wt, x)
                hit = real
            else:
                first = hit
                hit = hit | real
        pick = lambda a, c: torch.where(first[:, None] if a.dim() == 2 else first, a, c)  # noqa: E731
        vf, dr, eps, g, wt, x = (pick(a, c) for a, c in zip(keep, (vf, dr, eps, g, wt, x)))
        ch = (x[:, None] >= cum[g] + wt[:, None] * step[g]).sum(1).clamp(max=len(chans) - 1)
        inel = (kind[ch] == synth.EXCITATION) | (kind[ch] == synth.IONIZATION)
        real = hit & ~(inel & (eps < onset[ch]))
        us = _uniforms(k, 2, ids, seed)
        d = direction(us[0], us[1])
        sp = torch.sqrt((vf * vf).sum(1))
        cos = (d * vf).sum(1) / sp
        q = thr[ch] / eps
        root = torch.sqrt(torch.clamp(1.0 - q / c_m[ch], min=0.0))
        after = torch.where(inel, eps * (1.0 - c_m[ch] * q + c_ela[ch] * (root * cos - 1.0)), eps * (1.0 - c_ela[ch] * (1.0 - cos)))
        after = torch.where(kind[ch] == synth.ATTACHMENT, torch.zeros_like(after), torch.clamp(after, min=0.0))
        after = torch.where(kind[ch] == synth.IONIZATION, 0.5 * after, after)
        gi = gi + (real & (kind[ch] == synth.IONIZATION))
        da = da + (real & (kind[ch] == synth.ATTACHMENT))
        se, sep = torch.where(real, se + eps, se), torch.where(real, sep + after, sep)
        r = torch.where(real[:, None], r + dr, r)
        t = torch.where(real, t + flown, t)
        flown = torch.where(real, zero, flown)
        v = torch.where(real[:, None], c_speed * torch.sqrt(after)[:, None] * d, v)
        k = k + real
    return {"r": r, "t": t, "sum_eps": se, "sum_epsp": sep}, gi, da, k


def _stat(x):
    n = x.numel()
    sd = float(x.std()) if n > 1 else 0.0
    return [float(x.mean()), sd / math.sqrt(n), sd]


def exact(case, seed):
    if case["kind"] != "single" or case["precision"] != F64 or case["option"] != "plain":
        return None
    steps = case["collisions"] * max(1.0, 0.6 * _trials(case["gas"], case["td"]))
    if steps * max(1.0, case["electrons"] / 100_000.0) > 10_000:
        return None
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    rec, gi, da, k = _simulate(_config(case), case["electrons"], case["collisions"], int(seed), dev)
    r, t = rec["r"], rec["t"]
    v = r / t[:, None]
    zh = -r[:, 2]
    drift = [_stat(v[:, i]) for i in range(3)]
    drift = [[-drift[2][0]] + drift[2][1:]] + drift
    energy = [_stat(rec[n] / k) for n in ("sum_eps", "sum_epsp")]
    for e, n in zip(energy, ("sum_eps", "sum_epsp")):
        e[0] = float(rec[n].sum() / k.sum())
    mean = v.mean(0)
    diffusion, magnitude = [], []
    for m in (mean * torch.tensor([0.0, 0.0, 1.0], dtype=mean.dtype, device=dev), mean):
        x = r - t[:, None] * m
        z2, p2 = x[:, 2] ** 2, x[:, 0] ** 2 + x[:, 1] ** 2
        diffusion += [_stat((z2 + p2) / t), _stat(z2 / (2.0 * t)), _stat(p2 / (4.0 * t))]
        magnitude += [_stat(2.0 * torch.sqrt(z2 + p2)), _stat(2.0 * x[:, 2].abs()), _stat(2.0 * torch.sqrt(p2))]
    out = {"drift": drift, "energy": energy, "diffusion": diffusion, "magnitude": magnitude,
           "townsend": [_stat(gi / zh), _stat(da / zh)]}
    out = {n: np.array([a]) for n, a in out.items()}
    out["rates"] = np.array([[float(gi.sum() / zh.sum()), float(da.sum() / zh.sum())]])
    out.update({"efficiency": None, "majorant": None, "counts": None})
    if case["records"]:
        out.update({"rec_" + n: rec[n].cpu().numpy() for n in REALS})
        out["rec_ints"] = None
    return out
