"""The work this framework is used for, as cases that can be timed: lattices
stepped alone, batches, reduced-precision storage, the observation calls and
the serving loop, over the sizes that its workloads, tests and benchmark use.

  listed()            the cases
  draw(rng)           one more case of the same ranges
  prepare(case, seed) what a program holds before the call, on the GPU
  run(state)          one pass through the public entry points, its outputs
  work(case)          the bytes and operations one pass cannot do without
  exact(case, seed)   the outputs of the first pass in 64-bit torch, written
                      from the equations

Kinds of case.  "lattice": one lattice, `steps` time steps, then the state
(and the fields, with `fields`).  "batch": `count` lattices advanced together.
"observe": the diagnostics, the fields and a checkpoint written and read back,
between two short advances.  "serve": a burst of jobs through the server.
"""
import math

import numpy as np
import torch

from paper_2003_07968_amd import lbm
from paper_2003_07968_amd import workloads as W

DEV = "cuda" if torch.cuda.is_available() else "cpu"


def _case(name, kind, nx, ny, steps, storage="f64", shape="slab", tr=0.8, tau=1.0, sigma=1.0,
          collision="bgk", eos="unit", count=1, restart=False, fields=False, trace_alt=False):
    c = {"kind": kind, "nx": nx, "ny": ny, "steps": steps, "storage": storage, "shape": shape,
         "tr": tr, "tau": tau, "sigma": sigma, "collision": collision, "eos": eos, "count": count,
         "restart": restart, "fields": fields, "trace_alt": trace_alt}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest lattice in daily use (the reference run of the tests):
        # every launch is far too small to fill the chip, latency counts
        _case("droplet 64 f64", "lattice", 64, 64, 100, shape="droplet"),
        # the droplets behind the paper's tables and its oscillation runs: the
        # paper's equation of state, 200 x 200, with the MRT collision, sampled
        # every 100 steps
        _case("paper droplet 200 mrt f64", "lattice", 200, 200, 100, shape="droplet", tau=0.65,
              collision="mrt", eos="paper"),
        # ragged sides (strips and segments with remainders), an odd number of
        # steps: a short advance between two looks at the state
        _case("ragged 517x301 f64", "lattice", 517, 301, 21, shape="droplet", tr=0.75, tau=0.8,
              sigma=0.5),
        # the oscillating ellipse: the extent is read from the fields every 20
        # steps, so each short advance comes with a moments call
        _case("ellipse 1024 f64", "lattice", 1024, 1024, 20, shape="ellipse", tr=0.7, tau=0.8,
              fields=True),
        # the benchmark workload: four slabs at four temperatures as one batch,
        # in each storage mode
        _case("slabs 4x2048 f64", "batch", 2048, 2048, 100, count=4),
        _case("slabs 4x2048 f32", "batch", 2048, 2048, 100, "f32", count=4),
        # binary16 with one reference density loses mass over long runs, so
        # programs restart it from a checkpoint
        _case("slabs 4x2048 f16", "batch", 2048, 2048, 200, "f16", count=4, restart=True),
        _case("slabs 4x2048 f16l", "batch", 2048, 2048, 100, "f16l", count=4),
        # a parameter study: many uneven small droplets in one batch
        _case("study 48x[64,512] f32", "batch", 64, 512, 100, "f32", shape="droplet", count=48),
        # one large lattice (67 million cells)
        _case("slab 8192 f64", "lattice", 8192, 8192, 20),
        # steady-state criterion, fields, checkpoint and restart
        _case("observe 2048 f64", "observe", 2048, 2048, 4),
        # a burst of jobs through the serving loop, host buffers to host buffers
        _case("serve 12x[64,512] f32", "serve", 64, 512, 500, "f32", shape="droplet", count=12),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    storage = rng.choice(["f64", "f64", "f64", "f32", "f16", "f16l"])
    shape = rng.choice(["slab", "droplet", "droplet", "ellipse"])
    tr = round(rng.uniform(0.7, 0.9), 3)
    tau = round(rng.uniform(0.6, 1.2), 3)
    sigma = round(rng.uniform(0.25, 2.0), 3)
    coll = rng.choice(["bgk", "bgk", "mrt"])
    alt = rng.random() < 0.1
    kind = rng.choice(["lattice", "lattice", "lattice", "batch", "batch", "observe", "serve"])
    if kind == "lattice":
        nx, ny = log(24, 6000), log(24, 6000)
        top = int(8.0e8 / (nx * ny))  # cell updates of the largest listed cases: 1.3e9
        return _case(None, kind, nx, ny, max(1, min(log(1, 200), top)), storage, shape, tr, tau,
                     sigma, coll, restart=storage == "f16", fields=rng.random() < 0.3,
                     trace_alt=alt)
    if kind == "batch":
        if rng.random() < 0.5:  # equal lattices, the four temperatures in turn
            n = log(64, 1500)
            m = max(16, n + rng.randint(-16, 16))
            count = rng.randint(2, 8)
            steps = min(log(8, 120), int(8.0e8 / (count * n * m)))
            return _case(None, kind, n, m, steps, storage, "slab", tr, tau, sigma, coll,
                         count=count, restart=storage == "f16", trace_alt=alt)
        lo = log(32, 128)
        return _case(None, kind, lo, lo + log(32, 400), log(8, 150), storage, "droplet", tr, tau,
                     sigma, coll, count=rng.randint(3, 48), restart=storage == "f16",
                     trace_alt=alt)
    if kind == "observe":
        return _case(None, kind, log(32, 3000), log(32, 3000), rng.randint(1, 9), storage, shape,
                     tr, tau, sigma, coll, trace_alt=alt)
    lo = log(32, 128)
    return _case(None, kind, lo, lo + log(32, 400), log(50, 800), storage, "droplet", tr, tau,
                 sigma, coll, count=rng.randint(2, 12), trace_alt=alt)


# ---- inputs ----

def _field(p, shape, tr, eos, gen, frac=0.25):
    """The initial density of one lattice on the GPU: a slab, droplet or ellipse
    of Maxwell densities with seeded uniform noise of 1e-3."""
    nx, ny = p["nx"], p["ny"]
    rg, rl = W.PAPER_CS_MAXWELL[0.80] if eos == "paper" else W.unit_cs_coexistence(tr)
    width = 5.0 if eos == "paper" else 2.0
    x = torch.arange(nx, dtype=torch.float64, device=DEV)
    if shape == "slab":
        row = rg + 0.5 * (rl - rg) * (torch.tanh(2.0 * (x - (nx / 4.0 - 0.5)) / width)
                                      - torch.tanh(2.0 * (x - (3.0 * nx / 4.0 - 0.5)) / width))
        rho = row[None, :].repeat(ny, 1)
    else:
        y = torch.arange(ny, dtype=torch.float64, device=DEV)
        dx, dy = (x - (nx - 1) / 2.0)[None, :], (y - (ny - 1) / 2.0)[:, None]
        r0 = frac * min(nx, ny)
        ax, ay = (1.15 * r0, 0.87 * r0) if shape == "ellipse" else (r0, r0)
        r = torch.sqrt((dx / ax) ** 2 + (dy / ay) ** 2) * r0
        rho = 0.5 * (rl + rg) - 0.5 * (rl - rg) * torch.tanh(2.0 * (r - r0) / width)
    return rho + 1e-3 * (2.0 * torch.rand((ny, nx), dtype=torch.float64, device=DEV,
                                          generator=gen) - 1.0)


def _lattices(case, seed):
    """[(parameters, initial density)] of a case's lattices."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed) * 7919 + 17)
    host = np.random.default_rng(int(seed) * 104729 + 5)
    uneven = case["shape"] == "droplet" and case["count"] > 1
    out = []
    for k in range(case["count"]):
        nx, ny, tr, sigma, frac = case["nx"], case["ny"], case["tr"], case["sigma"], 0.25
        if uneven:  # sides over [nx, ny], the same for every seed; the rest is drawn
            t = (k * 0.618033988749895 + 0.5) % 1.0
            nx = ny = int(round(case["nx"] * (case["ny"] / case["nx"]) ** t))
            tr, frac = float(host.uniform(0.6, 0.9)), float(host.uniform(0.15, 0.35))
            sigma = float(host.uniform(0.25, 2.0))
        elif case["count"] > 1:
            tr = (0.6, 0.7, 0.8, 0.9)[k % 4]
        p = W.params(nx, ny, tr=tr, tau=case["tau"], sigma=sigma, eos=case["eos"],
                     m2_trace_alt=case["trace_alt"], storage=case["storage"],
                     collision=case["collision"], mrt=(1.0, 1.0, 1.0, 1.0, 1.0))
        rho0 = _field(p, case["shape"], tr, case["eos"], gen, frac)
        if case["storage"] in ("f32", "f16"):
            p["rho_ref"] = float(rho0.mean() if case["storage"] == "f32" else rho0.min())
        out.append((p, rho0))
    return out


def prepare(case, seed):
    items = _lattices(case, seed)
    st = {"case": case}
    if case["kind"] == "serve":
        need = sum(lbm.lbm_server_job_bytes(lbm.make_params(p), True) for p, _ in items)
        st["jobs"] = [(p, rho0.cpu().numpy(), case["steps"] + 37 * k)
                      for k, (p, rho0) in enumerate(items)]
        st["server"] = lbm.Server(need + (64 << 20), max_resident=64, quantum=64)
    elif case["kind"] == "batch":
        st["stream"] = torch.cuda.Stream()  # the batch replays graphs: not the null stream
        st["stream"].wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(st["stream"]):
            st["lats"] = [lbm.Lattice(p, rho0) for p, rho0 in items]
            st["batch"] = lbm.Batch(case["count"])
            for lat in st["lats"]:
                st["batch"].add(lat)
            if case["restart"]:
                st["f0"] = [lat.populations() for lat in st["lats"]]
        st["stream"].synchronize()
    else:
        (p, rho0), = items
        st["lat"] = lbm.Lattice(p, rho0)
        if case["restart"]:
            st["f0"] = st["lat"].populations()
    return st


def run(st):
    case = st["case"]
    n = case["steps"]
    if case["kind"] == "batch":
        with torch.cuda.stream(st["stream"]):
            if case["restart"]:
                for lat, f0 in zip(st["lats"], st["f0"]):
                    lat.set_populations(f0, 0)
            st["batch"].step(n)
            for lat in st["lats"]:
                lat.sync()
            return [lat.populations() for lat in st["lats"]]
    if case["kind"] == "serve":
        srv = st["server"]
        ids = [srv.submit(p, rho0, steps, want_populations=True) for p, rho0, steps in st["jobs"]]
        got = {}
        while len(got) < len(ids):
            srv.advance()
            for job, status, rho, f in srv.poll():
                got[job] = (status, rho, f)
        return [list(got[j]) for j in ids]
    lat = st["lat"]
    if case["restart"]:
        lat.set_populations(st["f0"], 0)
    if case["kind"] == "lattice":
        lat.step(n)
        lat.sync()
        out = {"f": lat.populations()}
        if case["fields"]:
            out["fields"] = lat.moments()
        return out
    # observe: advance, criterion and fields, checkpoint out and in, advance
    lat.step(n)
    d = lat.diagnostics()
    m = lat.moments()
    f = lat.populations()
    lat.set_populations(f, lat.t)
    lat.step(n)
    # (the net momentum is a sum that cancels to rounding: not an output)
    return {"diag": [d["mass"], d["ssc_num"], d["ssc_den"], d["umax"]], "fields": m, "f": f,
            "rho_after": lat.moments()["rho"]}


# ---- work ----

def _sizes(case):
    if case["shape"] == "droplet" and case["count"] > 1:
        side = [int(round(case["nx"] * (case["ny"] / case["nx"])
                          ** ((k * 0.618033988749895 + 0.5) % 1.0))) for k in range(case["count"])]
        return [s * s for s in side]
    return [case["nx"] * case["ny"]] * case["count"]


def work(case):
    """The state read and written once, however many steps; inputs and outputs
    in the form they are passed; about 160 operations per cell update (BGK), 230
    (MRT), as the kernels' arithmetic counts them."""
    state = {"f64": 72, "f32": 36, "f16": 18, "f16l": 22}[case["storage"]]
    ops = 160 if case["collision"] == "bgk" else 230
    cells, n = _sizes(case), case["steps"]
    if case["kind"] == "serve":  # density up; density and populations down
        steps = [n + 37 * k for k in range(case["count"])]
        return {"bytes": sum(c * (8 + 8 + 72) for c in cells),
                "flops": sum(c * s * ops for c, s in zip(cells, steps))}
    c = sum(cells)
    if case["kind"] == "observe":  # the state twice, snapshot, fields, checkpoint, density
        return {"bytes": c * (4 * state + 16 + 48 + 72 + 8), "flops": c * ops * (2 * n + 2)}
    extra = (72 if case["restart"] else 0) + (48 if case["fields"] else 0)
    return {"bytes": c * (2 * state + 72 + extra), "flops": c * ops * n}


# ---- 64-bit reference ----

_CX = (0, 1, 0, -1, 0, 1, -1, -1, 1)
_CY = (0, 0, 1, 0, -1, 1, 1, -1, -1)
_WT = (4 / 9,) + (1 / 9,) * 4 + (1 / 36,) * 4
# Gram-Schmidt moment matrix of D2Q9 (rho, e, zeta, j_x, q_x, j_y, q_y, p_xx, p_xy)
_M = ((1, 1, 1, 1, 1, 1, 1, 1, 1), (-4, -1, -1, -1, -1, 2, 2, 2, 2),
      (4, -2, -2, -2, -2, 1, 1, 1, 1), (0, 1, 0, -1, 0, 1, -1, -1, 1),
      (0, -2, 0, 2, 0, 1, -1, -1, 1), (0, 0, 1, 0, -1, 1, 1, -1, -1),
      (0, 0, -2, 0, 2, 1, 1, -1, -1), (0, 1, -1, 1, -1, 0, 0, 0, 0),
      (0, 0, 0, 0, 0, 1, -1, 1, -1))


def _equilibrium(rho, ux, uy):
    usq = ux * ux + uy * uy
    out = torch.empty((9,) + tuple(rho.shape), dtype=torch.float64, device=rho.device)
    for i in range(9):
        cu = _CX[i] * ux + _CY[i] * uy
        out[i] = _WT[i] * rho * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * usq)
    return out


def _fields(p, f):
    """rho, u, F and psi of the state f."""
    rho = f.sum(0)
    br = p["eos_b"] * rho
    P = p["eos_k"] * (p["eos_c"] * rho * p["T"] * (1 + br + br * br - br ** 3) / (1 - br) ** 3
                      - p["eos_a"] * rho * rho)
    psi = torch.sqrt((P - rho / 3.0) / p["G"])
    m0 = torch.zeros_like(psi)
    m1x, m1y, xx, yy, xy = (torch.zeros_like(psi) for _ in range(5))
    for i in range(9):
        s = _WT[i] * torch.roll(psi, (-_CY[i], -_CX[i]), (0, 1))
        m0 += s
        m1x += _CX[i] * s
        m1y += _CY[i] * s
        xx += (_CX[i] * _CX[i] - 1 / 3) * s
        yy += (_CY[i] * _CY[i] - 1 / 3) * s
        xy += _CX[i] * _CY[i] * s
    G, eps, sg = p["G"], p["epsilon"], p["sigma"]
    csc, ca, cb = -6.0 * G, 9.0 * G * (1.5 * eps - sg + 1.0), 9.0 * G * (sg - 1.0)
    tr = 2.0 / 3.0 * (m0 - psi) if p["m2_trace_alt"] else xx + yy
    Fx = csc * psi * m1x + ca * (m1x * xx + m1y * xy) + cb * m1x * tr
    Fy = csc * psi * m1y + ca * (m1x * xy + m1y * yy) + cb * m1y * tr
    jx = sum(_CX[i] * f[i] for i in range(9) if _CX[i])
    jy = sum(_CY[i] * f[i] for i in range(9) if _CY[i])
    return {"rho": rho, "ux": (jx + 0.5 * Fx) / rho, "uy": (jy + 0.5 * Fy) / rho, "Fx": Fx,
            "Fy": Fy, "psi": psi}


def _advance(p, f, steps):
    mrt = p["collision"] == W.COLLISION["mrt"]
    M = torch.tensor(_M, dtype=torch.float64, device=f.device)
    Mi = torch.linalg.inv(M.cpu()).to(f.device)
    lam = torch.tensor([1 / p[k] for k in ("tau_rho", "tau_e", "tau_zeta", "tau_j", "tau_q",
                                           "tau_j", "tau_q", "tau", "tau")],
                       dtype=torch.float64, device=f.device)
    A = Mi @ (lam[:, None] * M)
    B = Mi @ ((1 - lam / 2)[:, None] * M)
    om, g = 1.0 / p["tau"], 1.0 - 0.5 / p["tau"]
    for _ in range(steps):
        m = _fields(p, f)
        ux, uy, Fx, Fy = m["ux"], m["uy"], m["Fx"], m["Fy"]
        uF = ux * Fx + uy * Fy
        df = f - _equilibrium(m["rho"], ux, uy)
        S = torch.empty_like(f)
        for i in range(9):
            cF = _CX[i] * Fx + _CY[i] * Fy
            S[i] = _WT[i] * (3.0 * cF + 9.0 * cF * (_CX[i] * ux + _CY[i] * uy) - 3.0 * uF)
        if mrt:
            df, S = ((K @ v.reshape(9, -1)).reshape(v.shape) for K, v in ((A, df), (B, S)))
            f = f - df + S
        else:
            f = f - om * df + g * S
        f = torch.stack([torch.roll(f[i], (_CY[i], _CX[i]), (0, 1)) for i in range(9)])
    return f


def exact(case, seed):
    n, out = case["steps"], []
    for k, (p, rho0) in enumerate(_lattices(case, seed)):
        zero = torch.zeros_like(rho0)
        f = _advance(p, _equilibrium(rho0, zero, zero), n + (37 * k if case["kind"] == "serve"
                                                             else 0))
        if case["kind"] == "serve":
            out.append([None, f.sum(0).cpu().numpy(), f.cpu().numpy()])
        elif case["kind"] == "batch":
            out.append(f)
        elif case["kind"] == "lattice":
            out = {"f": f}
            if case["fields"]:
                out["fields"] = _fields(p, f)
        else:
            m = _fields(p, f)
            mass = float(m["rho"].sum())
            umax = float(torch.sqrt(m["ux"] ** 2 + m["uy"] ** 2).max())
            ssc = float((m["rho"] - rho0).abs().sum())
            out = {"diag": [mass, ssc, mass, umax], "fields": m, "f": f,
                   "rho_after": _fields(p, _advance(p, f, n))["rho"]}
    return out
