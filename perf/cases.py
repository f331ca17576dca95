"""Performance cases of the Monte Carlo lattice Boltzmann library on one GPU.

Each case is one piece of work as a program of this library does it, through
the public entry points of `paper_2608_23786_amd`. Five kinds:

* flow: draw an ensemble (init from Y), advance it, read the records and the
  whole velocity field of the final state;
* mixed: an ensemble of three resolutions (strides 16:4:1) with the velocity
  capture, the spectrum and structure function of every sample and the
  ensemble statistics at each save;
* gradient: the ensemble-mean kinetic energy after some steps and its gradient
  with respect to Y (forward with checkpoints, then the discrete adjoint);
* observables: spectrum and structure function of a resolution group, from its
  populations or from a velocity field in the capture's layout;
* statistics: what follows a campaign: 1-point Wasserstein distance, sample
  error, ensemble moments, dissipation rates in both forms, compensation.

Fields of an FP32 ensemble are kept as float32, the precision its populations
carry; everything of an FP64 ensemble and all FP64 post-processing stays
float64.

`exact` states each result in 64 bits with plain torch (its own lattice
Boltzmann step, FFTs and sorts), from the definitions alone.
"""
import itertools
import math

import numpy as np
import torch
from torch.utils.checkpoint import checkpoint

import paper_2608_23786_amd as mc
from paper_2608_23786_amd import ensemble as mce

DEVICE = "cuda:0"


def _flow(name, n, m, precision, ticks, *, re, u0, amp=0.05, project=True, lattice=27, stabiliser="closed_form",
          record_every=0, block=256, xcd_remap=0, buffer_addressing=1):
    return {"name": name, "kind": "flow", "n": n, "m": m, "precision": precision, "ticks": ticks, "re": re, "u0": u0,
            "amp": amp, "project": project, "lattice": lattice, "stabiliser": stabiliser,
            "record_every": record_every, "block": block, "xcd_remap": xcd_remap,
            "buffer_addressing": buffer_addressing}


def listed():
    return [
        # the smallest job: one plain Taylor-Green sample in FP64, 100 steps (launches and latency count)
        _flow("tgv32_f64", 32, 1, "f64", 100, re=100.0, u0=0.05, amp=0.0, project=False),
        # the ensemble the headline figure is quoted on: 64 samples of 64^3, records every 50 ticks
        _flow("rtgv64x64_f32", 64, 64, "f32s", 100, re=1600.0, u0=0.025, record_every=50),
        # a coarse rung of a sample-convergence study: many small samples, the D3Q19 lattice, odd tick counts
        _flow("set1000x32_d3q19_f32", 32, 1000, "f32s", 45, re=1280.0, u0=0.05, project=False, lattice=19,
              record_every=15),
        # a reference ensemble in FP64, an odd number of samples
        _flow("rtgv11x64_f64", 64, 11, "f64", 61, re=1600.0, u0=0.025, record_every=20),
        # the exact entropic stabiliser
        _flow("exact13x64_f32", 64, 13, "f32s", 40, re=1600.0, u0=0.025, stabiliser="exact", record_every=20),
        # one sample of the finest resolution of the vanishing-viscosity sequence, in its tuned launch shape
        _flow("rtgv1x512_f32", 512, 1, "f32s", 16, re=6400.0, u0=0.003125, block=512, xcd_remap=1,
              buffer_addressing=0),
        # the uneven batch: 64^3, 128^3 and 256^3 samples, observables and statistics at every save
        {"name": "mixed12_f32", "kind": "mixed", "n": 64, "m_coarse": 8, "m_mid": 3, "m_fine": 1, "saves": 2,
         "precision": "f32s", "lattice": 27},
        # the gradient workload, cut to 20 steps on two samples
        {"name": "gradient2x128_f32", "kind": "gradient", "n": 128, "m": 2, "precision": "f32s", "ticks": 20,
         "ckpt_every": 10, "re": 1600.0, "u0": 0.0125, "lattice": 27},
        # a small FP64 gradient, as a verification run or an optimiser on coarse samples takes it
        {"name": "gradient3x32_f64", "kind": "gradient", "n": 32, "m": 3, "precision": "f64", "ticks": 50,
         "ckpt_every": 10, "re": 100.0, "u0": 0.05, "lattice": 27},
        # spectrum and structure function of a resolution group straight from its populations, odd parity
        {"name": "observables12x128", "kind": "observables", "n": 128, "m": 12, "precision": "f32s", "lattice": 27,
         "from_velocity": False, "ticks": 3, "re": 3200.0, "u0": 0.0125},
        # the same from captured velocities at the resolution where a line no longer fits a wave
        {"name": "observables2x256_velocity", "kind": "observables", "n": 256, "m": 2, "precision": "f32s",
         "lattice": 27, "from_velocity": True, "ticks": 0, "re": 6400.0, "u0": 0.00625},
        # post-processing of a campaign of 1000 samples saved at 61 times
        {"name": "statistics1000", "kind": "statistics", "m": 1000, "q": 8, "n": 32, "nrec": 61},
    ]


# Node updates of the largest listed run (512^3, 16 ticks, FP32): what a drawn case may cost at most.
_MOST_UPDATES = 512 ** 3 * 16


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["flow", "flow", "flow", "flow", "mixed", "gradient", "observables", "observables", "statistics"])
    lattice = rng.choice([27, 27, 19])
    if kind == "flow":
        precision = rng.choice(["f32s", "f32s", "f64"])
        stabiliser = rng.choice(["closed_form", "closed_form", "closed_form", "exact"])
        n = rng.choice([8, 16, 32, 64, 64, 128, 256])
        dear = (2 if precision == "f64" else 1) * (4 if stabiliser == "exact" else 1)
        m = _log_int(rng, 1, max(1, min(1000, (1 << 25) // (dear * n ** 3))))
        ticks = _log_int(rng, 1, max(1, min(120, _MOST_UPDATES // (4 * dear * m * n ** 3))))
        every = rng.choice([0, 1 + ticks // 3, 1 + ticks // 2])
        c = _flow("", n, m, precision, ticks, re=rng.choice([100.0, 800.0, 25.0 * n]), u0=0.05 * 32.0 / max(n, 32),
                  amp=rng.choice([0.0, 0.025, 0.05]), project=rng.choice([True, False]), lattice=lattice,
                  stabiliser=stabiliser, record_every=every)
        # a seed has to give other inputs: without a perturbation it is the flow of one sample
        if c["amp"] == 0.0:
            c["amp"] = 0.1
    elif kind == "mixed":
        c = {"kind": "mixed", "n": rng.choice([32, 64]), "m_coarse": rng.randint(2, 9), "m_mid": rng.randint(2, 4),
             "m_fine": rng.randint(1, 2), "saves": rng.randint(1, 2), "precision": rng.choice(["f32s", "f64"]),
             "lattice": lattice}
    elif kind == "gradient":
        precision = rng.choice(["f32s", "f64"])
        n = rng.choice([8, 16, 32, 64, 128])
        m = _log_int(rng, 1, max(1, (1 << 22) // n ** 3))
        m = min(m, 64)
        ticks = _log_int(rng, 2, 40)
        c = {"kind": "gradient", "n": n, "m": m, "precision": precision, "ticks": ticks,
             "ckpt_every": rng.randint(1, ticks), "re": rng.choice([100.0, 1600.0]), "u0": 0.05 * 32.0 / max(n, 32),
             "lattice": lattice}
    elif kind == "observables":
        n = rng.choice([8, 16, 32, 64, 128, 256])
        m = _log_int(rng, 1, max(1, min(200, (1 << 25) // n ** 3)))
        c = {"kind": "observables", "n": n, "m": m, "precision": rng.choice(["f32s", "f64"]), "lattice": lattice,
             "from_velocity": rng.choice([True, False]), "ticks": rng.randint(0, 3), "re": 25.0 * n,
             "u0": 0.05 * 32.0 / max(n, 32)}
    else:
        c = {"kind": "statistics", "m": _log_int(rng, 3, 2000), "q": rng.choice([4, 8, 8, 16]),
             "n": rng.choice([16, 32]), "nrec": rng.randint(3, 90)}
    c.pop("name", None)
    return c


# ---------------------------------------------------------------- inputs
def _rng(seed):
    return np.random.default_rng([int(seed) & 0x7FFFFFFF, 2608])


def _draw_y(seed, m):
    return torch.from_numpy(_rng(seed).uniform(-1.0, 1.0, size=(m, 24)))


def _mixed_groups(case):
    n = case["n"]
    return [(n, case["m_coarse"], 16), (2 * n, case["m_mid"], 4), (4 * n, case["m_fine"], 1)]


def _mixed_flow(n):
    return 0.05 * 32.0 / n, 25.0 * n


def _u_fields(case, seed):
    """[m, 3, n, n, n]: Taylor-Green fields with random large-scale modes and small-scale noise, as a resolved run has."""
    n, m, u0 = case["n"], case["m"], case["u0"]
    g = torch.Generator(device=DEVICE).manual_seed(int(seed) & 0x7FFFFFFF)
    t = torch.arange(n, device=DEVICE, dtype=torch.float64) * (2 * math.pi / n)
    s, c = torch.sin(t), torch.cos(t)
    u = torch.empty((m, 3, n, n, n), dtype=torch.float64, device=DEVICE)
    for k in range(m):
        w = torch.randn(9, generator=g, dtype=torch.float64, device=DEVICE)
        u[k, 0] = c[:, None, None] * c[None, :, None] * s[None, None, :]
        u[k, 1] = -c[:, None, None] * s[None, :, None] * c[None, None, :]
        u[k, 2] = 0.05 * w[0] * torch.sin(2 * t)[:, None, None] * torch.cos(3 * t)[None, :, None] * s[None, None, :]
        u[k, 0] += 0.03 * w[1] * torch.sin(3 * t + w[2])[:, None, None] * torch.cos(2 * t + w[3])[None, :, None]
        u[k, 1] += 0.02 * w[4] * torch.cos(3 * t + w[5])[None, None, :] * torch.sin(2 * t)[:, None, None]
        u[k] += 1e-3 * torch.randn((3, n, n, n), generator=g, dtype=torch.float64, device=DEVICE)
    return u.mul_(u0)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "flow":
        s = mc.Sample(case["n"], case["u0"], case["re"], case["amp"], case["project"])
        ens = mc.Ensemble([s] * case["m"], case["precision"], lattice=case["lattice"])
        if case["stabiliser"] != "closed_form":
            ens.set_stabiliser(case["stabiliser"])
        if (case["block"], case["xcd_remap"], case["buffer_addressing"]) != (256, 0, 1):
            ens.set_launch(case["block"], case["xcd_remap"], case["buffer_addressing"], 1)
        y = _draw_y(seed, case["m"])
        if case["amp"] == 0.0:
            # without a perturbation Y does not enter: the viscosity of the run is what differs
            ens.set_viscosity([(1.0 + 0.1 * float(y[0, 0])) / case["re"]] * case["m"])
        return {"case": case, "ens": ens, "y": y}
    if kind == "mixed":
        samples, first, groups = [], 0, []
        for n, count, stride in _mixed_groups(case):
            u0, re = _mixed_flow(n)
            samples += [mc.Sample(n, u0, re, 0.05, True, stride)] * count
            groups.append((first, count))
            first += count
        ens = mc.Ensemble(samples, case["precision"], lattice=case["lattice"])
        vel = ens.capture_velocity()
        wb = max(int(mc.lib().mclbm_observables_range_work_bytes(ens._ctx, a, c)) for a, c in groups)
        with torch.cuda.stream(ens.stream):
            work = torch.empty(wb, dtype=torch.uint8, device=DEVICE)
        return {"case": case, "ens": ens, "y": _draw_y(seed, len(samples)), "groups": groups, "vel": vel, "work": work}
    if kind == "gradient":
        s = mc.Sample(case["n"], case["u0"], case["re"], 0.3, True)
        ens = mc.Ensemble([s] * case["m"], case["precision"], lattice=case["lattice"])
        return {"case": case, "ens": ens, "y": _draw_y(seed, case["m"]).to(DEVICE).requires_grad_()}
    if kind == "observables":
        s = mc.Sample(case["n"], case["u0"], case["re"], 0.05, True)
        ens = mc.Ensemble([s] * case["m"], case["precision"], lattice=case["lattice"])
        wb = int(mc.lib().mclbm_observables_range_work_bytes(ens._ctx, 0, case["m"]))
        with torch.cuda.stream(ens.stream):
            work = torch.empty(wb, dtype=torch.uint8, device=DEVICE)
        state = {"case": case, "ens": ens, "work": work}
        if case["from_velocity"]:
            state["u"] = _u_fields(case, seed)
        else:
            ens.init(y=_draw_y(seed, case["m"]))
            ens.step(case["ticks"])
        return state
    ens = mc.Ensemble([mc.Sample(case["n"], 0.05, 1280.0, 0.05, True)] * case["m"], "f32s", lattice=19)
    return dict(_statistics_inputs(case, seed), case=case, ens=ens)


def _statistics_inputs(case, seed):
    """Point values of two resolutions, and the energies, spectra and structure functions of a decaying turbulent run."""
    m, q3, n, nrec = case["m"], case["q"] ** 3, case["n"], case["nrec"]
    g = torch.Generator(device=DEVICE).manual_seed(int(seed) & 0x7FFFFFFF)

    def normal(*shape):
        return torch.randn(shape, generator=g, dtype=torch.float64, device=DEVICE)

    b = 0.5 * normal(1, 3, q3) + 0.1 * normal(m, 3, q3)
    a = b + 0.02 * normal(m, 3, q3)
    t = torch.linspace(0.0, 1.0, nrec, dtype=torch.float64, device=DEVICE)[:, None]
    u0 = 0.05
    ke = u0 ** 2 * 0.125 * torch.exp(-t * (1.0 + 0.1 * torch.rand((1, m), generator=g, dtype=torch.float64, device=DEVICE)))
    records = torch.zeros((nrec, m, 8), dtype=torch.float64, device=DEVICE)
    records[:, :, 0] = float(n ** 3)
    records[:, :, 4] = ke
    records[:, :, 5:] = 2.0 + 1e-3 * normal(nrec, m, 3)
    kappa = torch.arange(n // 2 + 1, dtype=torch.float64, device=DEVICE).clamp_min(1.0)
    shape = kappa ** (-5.0 / 3.0) / torch.sum(kappa ** (-5.0 / 3.0))
    ek = ke[:, :, None] * shape * torch.exp(0.05 * normal(1, m, n // 2 + 1))
    r = torch.arange(1, n // 2 + 1, dtype=torch.float64, device=DEVICE)
    s2 = u0 ** 2 * 0.1 * (r * (2 * math.pi / n)) ** (2.0 / 3.0) * torch.exp(0.05 * normal(m, n // 2))
    return {"a": a, "b": b, "records": records, "ek": ek.contiguous(), "s2": s2.contiguous()}


# ---------------------------------------------------------------- one pass
def _kept(case, t):
    """Results of an FP32 ensemble are kept in the precision it carries."""
    return t.float() if t is not None and case["precision"] == "f32s" else t


def run(state):
    case = state["case"]
    kind, ens = case["kind"], state["ens"]
    if kind == "flow":
        ens.init(y=state["y"])
        rec = ens.step(case["ticks"], record_every=case["record_every"])
        out = {}
        if rec is not None:
            out["records"] = _kept(case, rec)
        if case["m"] == 1:
            rho, u = ens.moments(0)
            out["rho"] = _kept(case, rho)
        else:
            u = ens.point_values(case["n"])   # every node is common to samples of one resolution
        out["u"] = _kept(case, u)
        return out
    if kind == "mixed":
        ens.init(y=state["y"])
        saves = []
        for _ in range(case["saves"]):
            rec = ens.step(16, record_every=16)[0]
            save = {"records": rec}
            for k, (first, count) in enumerate(state["groups"]):
                s2, ek = ens.observables_velocity_range(first, count, work=state["work"])
                many = count > 1
                ke_mean, ke_sd = mce.ensemble_moments(rec[first:first + count, 4:5], std=many)
                s2_mean, s2_sd = mce.ensemble_moments(s2, std=many)
                save.update({f"s2_{k}": s2, f"ek_{k}": ek, f"ke_mean_{k}": ke_mean, f"s2_mean_{k}": s2_mean})
                if many:
                    save.update({f"ke_sd_{k}": ke_sd, f"s2_sd_{k}": s2_sd})
            saves.append({k: _kept(case, v) for k, v in save.items()})
        return {"saves": saves, "u": _kept(case, state["vel"])}
    if kind == "gradient":
        j = mc.EnsembleKE.apply(state["y"], ens, case["ticks"], case["ckpt_every"])
        g, = torch.autograd.grad(j, state["y"])
        return {"J": _kept(case, j), "dJdY": _kept(case, g)}
    if kind == "observables":
        m = case["m"]
        if case["from_velocity"]:
            s2, ek = ens.observables_velocity_range(0, m, u=state["u"].view(-1), work=state["work"])
            return {"s2": s2, "ek": ek}
        s2, ek = ens.observables_range(0, m, work=state["work"])
        return {"s2": _kept(case, s2), "ek": _kept(case, ek)}
    a, b, q = state["a"], state["b"], case["q"]
    records, ek, s2 = state["records"], state["ek"], state["s2"]
    mid = case["nrec"] // 2
    d, eta = ens.dissipation(records, 0, 10)
    ds, etas = ens.dissipation_spectra(0, ek, 0, 10)
    s2c, ekc = ens.compensate(0, d[mid], s2, ek[mid])
    s2_mean, s2_sd = mce.ensemble_moments(s2)
    ek_mean, ek_sd = mce.ensemble_moments(ek[mid])
    ke_mean, ke_sd = mce.ensemble_moments(records[mid, :, 4:5])
    return {"w1": mce.w1_1pt(a, b, q), "error": mce.sample_error(a, b, q), "d": d, "eta": eta, "ds": ds, "etas": etas,
            "s2c": s2c, "ekc": ekc, "s2_mean": s2_mean, "s2_sd": s2_sd, "ek_mean": ek_mean, "ek_sd": ek_sd,
            "ke_mean": ke_mean, "ke_sd": ke_sd}


# ---------------------------------------------------------------- what a pass cannot do without
# Additions and multiplications of one node update, counted from the formulas:
# moments (q + 3 * 2q/3), equilibrium (6q), non-equilibrium part (q), its six
# second moments (~3q), the two inner products (5q with one reciprocal per
# population), the relaxed state (4q). The exact stabiliser adds at least one
# Newton step (a logarithm, a reciprocal and 8 operations per population).
def _update_flops(q, exact=False):
    return 22 * q + (20 * q if exact else 0)


def _fft_flops(n):
    # four half-spectrum 3-D real transforms (three components, one inverse), 2.5 N log2 N each
    return 4 * 2.5 * n ** 3 * 3 * math.log2(n)


def work(case):
    """Inputs read once, outputs written once, the populations of the state read and written once per pass."""
    kind = case["kind"]
    if kind == "statistics":
        m, q3, n, nrec = case["m"], case["q"] ** 3, case["n"], case["nrec"]
        rows = m * (n + 1)
        return {"bytes": 8.0 * (2 * m * 3 * q3 + nrec * m * (1 + n // 2 + 1 + 2) + 3 * rows),
                "flops": 3.0 * q3 * m * (2 * math.log2(max(2, m)) + 12) + nrec * m * (n // 2 + 10) + 40.0 * rows}
    e = 8 if case["precision"] == "f64" else 4
    q = case["lattice"]
    if kind == "observables":
        nodes = case["m"] * case["n"] ** 3
        return {"bytes": float(nodes) * (24 if case["from_velocity"] else q * e) + 8.0 * case["m"] * (case["n"] + 1),
                "flops": case["m"] * _fft_flops(case["n"])}
    if kind == "mixed":
        bytes_, flops = 0.0, 0.0
        for n, count, stride in _mixed_groups(case):
            nodes = float(count) * n ** 3
            bytes_ += nodes * (2 * q * e + 24 * case["saves"])
            flops += nodes * case["saves"] * 16 // stride * _update_flops(q) + count * case["saves"] * _fft_flops(n)
        return {"bytes": bytes_, "flops": flops}
    nodes = float(case["m"]) * case["n"] ** 3
    if kind == "gradient":
        # the states are needed again in reverse order: each is written once and read once
        return {"bytes": nodes * (2 * q * e) * case["ticks"], "flops": nodes * case["ticks"] * 4 * _update_flops(q)}
    return {"bytes": nodes * (2 * q * e + 3 * e),
            "flops": nodes * case["ticks"] * _update_flops(q, case["stabiliser"] == "exact")}


# ---------------------------------------------------------------- the same results in 64 bits
class _Lattice:
    def __init__(self, q):
        c = [v for v in itertools.product((-1, 0, 1), repeat=3) if q == 27 or sum(map(abs, v)) < 3]
        w = {27: {0: 8 / 27, 1: 2 / 27, 2: 1 / 54, 3: 1 / 216}, 19: {0: 1 / 3, 1: 1 / 18, 2: 1 / 36}}[q]
        self.c = c
        self.cm = torch.tensor(c, dtype=torch.float64, device=DEVICE)                      # [q, 3]
        self.w = torch.tensor([w[sum(map(abs, v))] for v in c], dtype=torch.float64, device=DEVICE)[:, None]
        kind = self.cm.abs().sum(1)
        x, y, z = self.cm.unbind(1)
        face, edge = (kind == 1).double(), (kind == 2).double()
        # second moments of the non-equilibrium part: xx - zz, yy - zz, xy, xz, yz
        self.to_p = torch.stack([x * x - z * z, y * y - z * z, x * y, x * z, y * z])
        # the population vector that carries those moments and no others
        self.shear = torch.stack([face * (2 * x * x - y * y - z * z) / 6, face * (2 * y * y - x * x - z * z) / 6,
                                  edge * x * y / 4, edge * x * z / 4, edge * y * z / 4], dim=1)     # [q, 5]


def _collide(lat, g, nu, exact):
    """Post-collision populations minus the weights of [q, cells] populations minus the weights."""
    omega = 1.0 / (3.0 * nu + 0.5)
    drho = g.sum(0)
    j = lat.cm.T @ g
    rho = 1.0 + drho
    u = j / rho
    cu = lat.cm @ u
    geq = lat.w * (drho + 3.0 * (lat.cm @ j) + rho * (4.5 * cu * cu - 1.5 * (u * u).sum(0)))
    fneq = g - geq
    ds = lat.shear @ (lat.to_p @ fneq)
    dh = fneq - ds
    r = 1.0 / (lat.w + geq)
    a, b = (ds * dh * r).sum(0), (dh * dh * r).sum(0)
    active = b > 1e-26     # dh is rounding below: the populations do not depend on gamma there
    safe = torch.where(active, b, torch.ones_like(b))
    gamma = torch.where(active, 2.0 / omega - (2.0 - 2.0 / omega) * a / safe, torch.full_like(b, 2.0))
    t = 0.5 * omega * gamma
    if exact:
        base = g - omega * ds
        for _ in range(8):
            f = lat.w + base - t * dh
            d1 = (dh * (torch.log1p((base - t * dh) / lat.w) - 3.0 * cu)).sum(0)
            d2 = (dh * dh / f).sum(0)
            t = torch.where(active, t + d1 / torch.where(active, d2, torch.ones_like(d2)), t)
        gamma = 2.0 * t / omega
    return g - omega * ds - t * dh, (drho, j, u, gamma)


def _stream(lat, g, n):
    g = g.view(len(lat.c), n, n, n)
    return torch.stack([torch.roll(g[i], (c[2], c[1], c[0]), (0, 1, 2)) for i, c in enumerate(lat.c)]).view(len(lat.c), -1)


def _initial(lat, y, n, u0, amp, project):
    """Initial equilibrium of the (projected) randomised Taylor-Green field; y: [24]."""
    t = torch.arange(n, device=DEVICE, dtype=torch.float64) * (2 * math.pi / n)
    s, c = torch.sin(t), torch.cos(t)
    one = torch.ones(n, dtype=torch.float64, device=DEVICE)
    tgv = torch.stack([torch.einsum("z,y,x->zyx", c, c, s), -torch.einsum("z,y,x->zyx", c, s, c),
                       0.0 * torch.einsum("z,y,x->zyx", one, one, one)])
    basis = torch.stack([torch.sin(2 * t), torch.cos(2 * t)])
    coef = y.view(3, 2, 2, 2)
    p = (coef.reshape(12, 2) @ basis).view(3, 2, 2, n)                                   # over k: [a, i, j, z]
    p = (p.permute(0, 1, 3, 2).reshape(-1, 2) @ basis).view(3, 2, n, n)                  # over j: [a, i, z, y]
    p = 0.125 * (p.permute(0, 2, 3, 1).reshape(-1, 2) @ basis).view(3, n, n, n)          # over i: [a, z, y, x]
    if project:
        k = torch.fft.fftfreq(n, 1.0 / n, dtype=torch.float64, device=DEVICE)
        kx, ky, kz = k[None, None, :], k[None, :, None], k[:, None, None]
        k2 = (kx * kx + ky * ky + kz * kz).clamp_min(1.0)
        ph = torch.fft.fftn(p, dim=(1, 2, 3))
        div = (kx * ph[0] + ky * ph[1] + kz * ph[2]) / k2
        p = torch.fft.ifftn(torch.stack([ph[0] - kx * div, ph[1] - ky * div, ph[2] - kz * div]), dim=(1, 2, 3)).real
    u = (u0 * (tgv + amp * p)).reshape(3, -1)
    cu = lat.cm @ u
    return lat.w * (3.0 * cu + 4.5 * cu * cu - 1.5 * (u * u).sum(0))


def _record(g, parts):
    drho, j, u, gamma = parts
    n3 = drho.numel()
    return torch.stack([n3 + drho.sum(), j[0].sum(), j[1].sum(), j[2].sum(), 0.5 * (u * u).sum() / n3, gamma.min(),
                        gamma.max(), gamma.mean()])


def _velocity(lat, g):
    return (lat.cm.T @ g) / (1.0 + g.sum(0))


def _observables(u):
    """S2(r) and E(kappa) of one velocity field [3, n, n, n]."""
    n = u.shape[-1]
    k = torch.fft.fftfreq(n, 1.0 / n, dtype=torch.float64, device=DEVICE)
    length2 = k[:, None, None] ** 2 + k[None, :, None] ** 2 + k[None, None, :] ** 2
    shell = torch.round(torch.sqrt(length2)).long().view(-1)
    psi = torch.zeros((n, n, n), dtype=torch.float64, device=DEVICE)
    for a in range(3):
        f = torch.fft.fftn(u[a])
        psi += f.real ** 2 + f.imag ** 2
    r = torch.fft.ifftn(psi).real / n ** 3
    top = int(shell.max()) + 1
    size = torch.bincount(shell, minlength=top).double()

    def sums(v):
        return torch.zeros(top, dtype=torch.float64, device=DEVICE).index_add_(0, shell, v.reshape(-1))

    ek = 4 * math.pi / size * sums(0.5 * length2 * psi) / float(n) ** 6
    s2 = sums(2.0 * (r[0, 0, 0] - r)) / size
    return s2[1:n // 2 + 1], ek[:n // 2 + 1]


def _moments(x):
    return x.mean(0), x.std(0) if x.shape[0] > 1 else None


def _exact_flow(case, seed):
    n, m, q = case["n"], case["m"], case["lattice"]
    if m * n ** 3 * case["ticks"] * (6 if case["stabiliser"] == "exact" else 1) > 4.0e9 or n > 256:
        return None
    lat, y = _Lattice(q), _draw_y(seed, m).to(DEVICE)
    every, exact = case["record_every"], case["stabiliser"] == "exact"
    us, recs = [], []
    for s in range(m):
        re = case["re"] / (1.0 + 0.1 * float(y[0, 0])) if case["amp"] == 0.0 else case["re"]
        nu = case["u0"] * n / (2 * math.pi * re)
        g = _initial(lat, y[s], n, case["u0"], case["amp"], case["project"])
        rec = []
        for t in range(case["ticks"]):
            out, parts = _collide(lat, g, nu, exact)
            if every and t % every == 0:
                rec.append(_record(g, parts))
            g = _stream(lat, out, n)
        us.append(_velocity(lat, g))
        recs.append(torch.stack(rec) if rec else None)
    out = {}
    if every:
        out["records"] = torch.stack(recs, dim=1)
    if m == 1:
        out["rho"] = (1.0 + g.sum(0)).view(n, n, n)
        out["u"] = us[0].view(3, n, n, n)
    else:
        out["u"] = torch.stack(us)
    return out


def _exact_mixed(case, seed):
    lat = _Lattice(case["lattice"])
    groups = _mixed_groups(case)
    y = _draw_y(seed, sum(c for _, c, _ in groups)).to(DEVICE)
    saves = [dict(records=None) for _ in range(case["saves"])]
    vel, s = [], 0
    for k, (n, count, stride) in enumerate(groups):
        u0, re = _mixed_flow(n)
        rows = [([], [], []) for _ in range(case["saves"])]
        for _ in range(count):
            g = _initial(lat, y[s], n, u0, 0.05, True)
            for save in range(case["saves"]):
                for _ in range(16 // stride if save else 0):
                    out, _parts = _collide(lat, g, u0 * n / (2 * math.pi * re), False)
                    g = _stream(lat, out, n)
                u = _velocity(lat, g)
                s2, ek = _observables(u.view(3, n, n, n))
                for row, v in zip(rows[save], (s2, ek, 0.5 * (u * u).sum() / n ** 3)):
                    row.append(v)
            vel.append(u.reshape(-1))
            s += 1
        for save, (s2, ek, ke) in zip(saves, rows):
            s2, ek, ke = torch.stack(s2), torch.stack(ek), torch.stack(ke)[:, None]
            save.update({f"s2_{k}": s2, f"ek_{k}": ek})
            for word, v in (("ke", ke), ("s2", s2)):
                mean, sd = _moments(v)
                save[f"{word}_mean_{k}"] = mean
                if count > 1:
                    save[f"{word}_sd_{k}"] = None   # a difference of nearly equal numbers in an FP32 run
    return {"saves": saves, "u": torch.cat(vel)}


def _exact_gradient(case, seed):
    n, m = case["n"], case["m"]
    if m * n ** 3 * case["ticks"] > 3.0e8:
        return None
    lat, y = _Lattice(case["lattice"]), _draw_y(seed, m).to(DEVICE)
    nu = case["u0"] * n / (2 * math.pi * case["re"])

    def step(g):
        return _stream(lat, _collide(lat, g, nu, False)[0], n)

    total, grads = 0.0, []
    for s in range(m):
        ys = y[s].clone().requires_grad_()
        g = _initial(lat, ys, n, case["u0"], 0.3, True)
        for _ in range(case["ticks"]):
            g = checkpoint(step, g, use_reentrant=False)
        u = _velocity(lat, g)
        j = 0.5 * (u * u).sum() / n ** 3 / m
        grads.append(torch.autograd.grad(j, ys)[0])
        total = total + j.detach()
    return {"J": total, "dJdY": torch.stack(grads)}


def _exact_observables(case, seed):
    n, m = case["n"], case["m"]
    if case["from_velocity"]:
        rows = [_observables(u) for u in _u_fields(case, seed)]
    else:
        lat, y, rows = _Lattice(case["lattice"]), _draw_y(seed, m).to(DEVICE), []
        for s in range(m):
            g = _initial(lat, y[s], n, case["u0"], 0.05, True)
            for _ in range(case["ticks"]):
                g = _stream(lat, _collide(lat, g, case["u0"] * n / (2 * math.pi * case["re"]), False)[0], n)
            rows.append(_observables(_velocity(lat, g).view(3, n, n, n)))
    return {"s2": torch.stack([r[0] for r in rows]), "ek": torch.stack([r[1] for r in rows])}


def _exact_statistics(case, seed):
    i = _statistics_inputs(case, seed)
    a, b, records, ek, s2 = i["a"], i["b"], i["records"], i["ek"], i["s2"]
    m, n, nrec, q3, mid = case["m"], case["n"], case["nrec"], case["q"] ** 3, case["nrec"] // 2
    u0, every = 0.05, 10
    w1 = (torch.sort(a, dim=0).values - torch.sort(b, dim=0).values).abs().mean(0).sum(1) / q3
    num = [(a[:, c] - b[:, c]).abs().sum(1) for c in range(3)] + [(a - b).square().sum(1).sqrt().sum(1)]
    den = [b[:, c].abs().sum(1) for c in range(3)] + [b.square().sum(1).sqrt().sum(1)]
    error = torch.stack([(x / z).mean() for x, z in zip(num, den)])
    t = torch.arange(nrec, dtype=torch.float64, device=DEVICE)[:, None] * every * (2 * math.pi / n) * u0

    def rate(energy):
        lo = torch.arange(nrec, device=DEVICE).sub(1).clamp_min(0)
        hi = torch.arange(nrec, device=DEVICE).add(1).clamp_max(nrec - 1)
        d = -(energy[hi] - energy[lo]) / u0 ** 2 / (t[hi] - t[lo])
        return d, ((1.0 / 1280.0) ** 3 / d.mean(1)) ** 0.25

    d, eta = rate(records[:, :, 4])
    ds, etas = rate(ek.sum(2))
    kappa = torch.arange(n // 2 + 1, dtype=torch.float64, device=DEVICE)
    lag = torch.arange(1, n // 2 + 1, dtype=torch.float64, device=DEVICE) * (2 * math.pi / n)
    dm = d[mid][:, None]
    out = {"w1": w1, "error": error, "d": d, "eta": eta, "ds": ds, "etas": etas,
           "s2c": s2 / u0 ** 2 / (dm * lag) ** (2 / 3),
           "ekc": kappa ** (5 / 3) * ek[mid] / u0 ** 2 / (1.5 * dm ** (2 / 3))}
    for word, v in (("s2", s2), ("ek", ek[mid]), ("ke", records[mid, :, 4:5])):
        out[f"{word}_mean"], out[f"{word}_sd"] = _moments(v)
    return out


def exact(case, seed):
    return {"flow": _exact_flow, "mixed": _exact_mixed, "gradient": _exact_gradient, "observables": _exact_observables,
            "statistics": _exact_statistics}[case["kind"]](case, seed)
