"""The workloads whose speed is measured, through the package's public calls.

A case is a dict of plain values; `kind` says which path it takes:

  poisson   one field solve of a given charge density (Sim.poisson)
  langmuir  a Langmuir wave of one species in a periodic box: a run of steps,
            then the field, the densities and the phase space
  argon     one argon RF discharge or a batch of them (bounded gap, walls,
            secondary emission, collisions, births), with or without the time
            averages: a run of steps, then the profiles and the counters
  box       the E x B drift box of electrons and xenon ions (periodic,
            magnetised), with or without axial renewal
  swarm     electron swarms at several E/N with ionization, thinned on the
            device between runs of steps
  train     Adam steps of the warm-start network on minibatches
  forward   the warm-start network's prediction

`listed` names the sizes the package's own drivers, tests and benchmark use,
from the smallest call to the largest; `draw` gives other sizes of the same
ranges.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import workloads as W

HOST_LOADED = 4_500_000        # particles per species up to which the inputs are made here and handed over
EN_TD = (50.0, 100.0, 200.0, 500.0, 1000.0)


def listed():
    return [
        # one field solve of the argon gap's mesh for a density the caller holds: the smallest call
        dict(name="poisson_gap", kind="poisson", cells=400, bounded=True),
        # the Langmuir wave of the paper's worked example (65,536 electrons): a short run and its phase space
        dict(name="langmuir_wave", kind="langmuir", n=65536, cells=128, steps=512),
        # one argon discharge with the library's own schedule and time averages on, one RF period
        dict(name="argon_sampled", kind="argon", batch=1, total=400006, cells=400, sampled=True, schedule="default",
             steps=1600),
        # one argon discharge on its way to its steady state (no averages), with the schedule the autotuner takes
        dict(name="argon_relaxing", kind="argon", batch=1, total=400000, cells=400, sampled=False, schedule="256",
             steps=1600),
        # a batched sweep of 64 discharges that takes its averages as it runs
        dict(name="sweep_sampled", kind="argon", batch=64, total=17700000, cells=0, sampled=True, schedule="default",
             steps=128),
        # the same sweep at its full steady-state counts (4.9e7 particles), no averages, autotuned schedule
        dict(name="sweep_full", kind="argon", batch=64, total=49000000, cells=0, sampled=False, schedule="1024",
             steps=64),
        # the E x B box of the benchmark: 4e6 electrons and 4e6 xenon ions on 1024 cells
        dict(name="exb_box", kind="box", n=4000000, cells=1024, steps=256, renew=False),
        # the same box with eight times the particles, beyond every cache
        dict(name="exb_box_large", kind="box", n=32000000, cells=1024, steps=32, renew=False),
        # the electron cyclotron drift box with axial renewal, between two of its density samples
        dict(name="ecdi_box", kind="box", n=4000000, cells=1024, steps=128, renew=True),
        # forty electron swarms (five E/N, eight replicas each) between two thinnings
        dict(name="swarm", kind="swarm", replicas=8, n=100000, steps=128),
        # training the warm-start network: minibatches of 64
        dict(name="train", kind="train", hidden=256, batch=64, steps=64),
        # its prediction for as many parameter sets as a model holds at once
        dict(name="forward", kind="forward", hidden=256, batch=4096),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["poisson", "langmuir", "argon", "argon", "box", "swarm", "train", "forward"])
    if kind == "poisson":
        return dict(kind=kind, cells=_log_int(rng, 16, 4095), bounded=rng.random() < 0.6)
    if kind == "langmuir":
        return dict(kind=kind, n=_log_int(rng, 1000, 1000000), cells=_log_int(rng, 32, 1024),
                    steps=rng.choice([96, 200, 256, 384]))
    if kind == "argon":
        batch = 1 if rng.random() < 0.5 else rng.randint(2, 64)
        total = _log_int(rng, 2e4, 4e6) if batch == 1 else batch * _log_int(rng, 4e4, 3e5)
        return dict(kind=kind, batch=batch, total=total, cells=rng.randint(200, 600) if batch == 1 else 0,
                    sampled=rng.random() < 0.5, schedule=rng.choice(["default", "256", "1024"]),
                    steps=rng.choice([128, 200, 320]))
    if kind == "box":
        return dict(kind=kind, n=_log_int(rng, 1e5, 1.2e7), cells=_log_int(rng, 128, 2048),
                    steps=rng.choice([32, 64, 100]), renew=rng.random() < 0.4)
    if kind == "swarm":
        return dict(kind=kind, replicas=rng.randint(1, 8), n=_log_int(rng, 1e4, 1e5), steps=rng.choice([64, 128]))
    if kind == "train":
        return dict(kind=kind, hidden=rng.choice([64, 96, 128, 200, 256, 384]), batch=_log_int(rng, 16, 512),
                    steps=rng.choice([8, 16, 32]))
    return dict(kind=kind, hidden=rng.choice([64, 96, 128, 200, 256, 384]), batch=_log_int(rng, 1, 4096))


# ---- inputs -----------------------------------------------------------------
def _widths(case):
    h = case["hidden"]
    return (W.WARM_WIDTHS[0], h, h, h, W.WARM_WIDTHS[-1])


def _box_config(case, seed):
    if case["kind"] == "langmuir":
        return W.langmuir(k_lambda=0.38, n_cells=case["cells"], n_particles=case["n"], eps=0.02, seed=1 + seed)
    length = 15 * W.lambda1() if case["renew"] else 0.005
    cfg = W.exb(length=length, n_cells=case["cells"], n_per_species=case["n"],
                density=1e17 if case["renew"] else 5e16, seed=1 + seed)
    if case["renew"]:
        cfg["renew_lz"] = 0.01
    return cfg


def _box_particles(cfg, seed):
    """Stratified positions (in cells; a density wave where the configuration
    asks for one) and drifting Maxwellians of every species, on the GPU."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000 + seed)
    nc = cfg["n_cells"]
    out = []
    for sp in cfg["species"]:
        n = sp["n_init"]
        u = torch.rand(n, generator=gen, device="cuda", dtype=torch.float64)
        x = (torch.arange(n, device="cuda", dtype=torch.float64) + u) / n
        if cfg["perturb_eps"]:
            k = 2.0 * math.pi * cfg["perturb_mode"]
            x = torch.remainder(x - cfg["perturb_eps"] / k * torch.sin(k * x), 1.0)
        x = x * nc
        cell = torch.clamp(x.floor(), max=nc - 1)
        off = torch.clamp((x - cell).float(), max=1.0 - 2.0 ** -24)
        v = torch.randn((3, n), generator=gen, device="cuda", dtype=torch.float64) * sp["vth"]
        v += torch.tensor(sp["drift"], device="cuda", dtype=torch.float64)[:, None]
        out.append(dict(cell=cell.int(), off=off, v=v.float()))
    return out


def _network_params(widths, seed):
    rng = np.random.default_rng(seed)
    blocks = []
    for a, b in zip(widths[:-1], widths[1:]):
        w = np.zeros((b, a + 1))
        w[:, :a] = rng.normal(0.0, math.sqrt(2.0 / a), (b, a))
        blocks.append(w.ravel())
    return np.concatenate(blocks).astype(np.float32)


def _network_batches(case, seed):
    """Scaled discharge parameters in [0, 1] and standardised profiles that
    depend smoothly on them."""
    rng = np.random.default_rng(7000 + seed)
    n_in, n_out = W.WARM_WIDTHS[0], W.WARM_WIDTHS[-1]
    m = case["batch"] * min(case.get("steps", 1), 16)
    x = rng.uniform(0.0, 1.0, (m, n_in))
    grid = np.linspace(0.0, 1.0, n_out)
    phase = x @ rng.uniform(-2.0, 2.0, (n_in, 3))
    t = np.sin(2.0 * math.pi * grid + phase[:, :1]) + 0.5 * np.cos(5.0 * grid + phase[:, 1:2]) * phase[:, 2:]
    return x.astype(np.float32), (t / t.std()).astype(np.float32)


def _charge_density(case, seed):
    nodes = case["cells"] + (1 if case["bounded"] else 0)
    rng = np.random.default_rng(500 + seed)
    x = np.linspace(0.0, 1.0, nodes)
    return W.E_CHARGE * 1e15 * (np.cos(math.pi * x) ** 8 + 0.05 * rng.normal(0.0, 1.0, nodes))


def _gap_config(case):
    if case["bounded"]:
        return W.argon_rf(n_cells=case["cells"], n_init=1000, capacity=4096)
    return W.exb(n_cells=case["cells"], n_per_species=1000, capacity=4096)


def _argon_sim(P, case, seed):
    batch = case["batch"]
    if batch == 1:
        n = np.array([case["total"] // 2])
        cfgs = [W.argon_rf(n_cells=case["cells"], capacity=4 * int(n[0]) + 65536, seed=1 + seed)]
    else:
        draws = W.sweep_draws(batch, seed=4)
        full = W.steady_counts(batch)
        n = np.maximum(1000, np.rint(full * (case["total"] / (2.0 * full.sum())))).astype(int)
        weight = W.PILOT_WEIGHT * full / n           # every discharge keeps its densities
        cfgs = [W.argon_rf(gap=d["gap"], n_cells=d["n_cells"], pressure_mtorr=d["pressure_mtorr"], v_amp=d["v_amp"],
                           seed=1000 * (1 + seed) + i, capacity=4 * int(n[i]) + 65536, weight=float(weight[i]))
                for i, d in enumerate(draws)]
    for cfg in cfgs:
        for sp in cfg["species"]:
            sp["load"], sp["n_init"] = W.LOAD_NONE, 0
    sim = P.Sim(cfgs, W.argon_tables())
    dens, temp = W.discharge_profile()
    for b in range(batch):
        sim.load_profiles(dens, temp, [int(n[b]), int(n[b])], batch=b)
    if case["schedule"] == "256":
        sim.config_tiles(4, 256, 0, 32)
        sim.config_events(True)
    elif case["schedule"] == "1024":
        sim.config_tiles(4, 1024, 0, 32)
    if case["sampled"]:
        sim.set_diag(True)
    return sim


def prepare(case, seed):
    import paper_2609_17151_amd as P
    kind = case["kind"]
    if kind == "poisson":
        return dict(case=case, sim=P.Sim(_gap_config(case)), rho=_charge_density(case, seed), t=1e-9)
    if kind in ("langmuir", "box"):
        cfg = _box_config(case, seed)
        if case["n"] <= HOST_LOADED:
            empty = dict(cfg, species=[dict(sp, load=W.LOAD_NONE, n_init=0) for sp in cfg["species"]])
            sim = P.Sim(empty)
            for s, p in enumerate(_box_particles(cfg, seed)):
                cell, off, v = (p[k].cpu().numpy() for k in ("cell", "off", "v"))
                sim.set_particles(s, cell, off, v[0], v[1], v[2], np.arange(len(cell), dtype=np.uint32), len(cell), 0)
        else:
            sim = P.Sim(cfg)
        return dict(case=case, sim=sim)
    if kind == "argon":
        return dict(case=case, sim=_argon_sim(P, case, seed))
    if kind == "swarm":
        from paper_2609_17151_amd.swarm import Swarm
        sw = Swarm(EN_TD, replicas=case["replicas"], n=case["n"], seed=1 + 100000 * seed)
        return dict(case=case, sim=sw.sim, above=int(sw.control * sw.n0), keep=sw.n0)
    widths = _widths(case)
    net = P.MLP(widths, max(case["batch"], 16))
    net.set_params(_network_params(widths, seed))
    x, t = (torch.from_numpy(a).cuda() for a in _network_batches(case, seed))
    b = case["batch"]
    if kind == "forward":
        return dict(case=case, net=net, x=x[:b])
    sets = [(x[i:i + b], t[i:i + b]) for i in range(0, len(x), b)]
    return dict(case=case, net=net, sets=sets, losses=torch.zeros(case["steps"], dtype=torch.float32, device="cuda"))


# ---- one pass ------------------------------------------------------------------
def _counts(sim):
    rows = [sim.counts(b) for b in range(sim.B)]
    return np.array([[r["step"], r["flags"]] + r["count"] + r["next_id"] for r in rows], dtype=np.int64)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "poisson":
        phi, ef = state["sim"].poisson(state["t"], state["rho"])
        return dict(phi=phi, efield=ef)
    if kind == "forward":
        return dict(y=state["net"].forward(state["x"]))
    if kind == "train":
        net, sets, losses = state["net"], state["sets"], state["losses"]
        for k in range(case["steps"]):
            x, t = sets[k % len(sets)]
            net.train_step(x, t, lr=1e-3, loss_out=losses[k:k + 1])
        return dict(losses=losses, params=net.params())
    sim = state["sim"]
    sim.step(case["steps"])
    if kind == "swarm":
        sim.thin(0, state["above"], state["keep"])
        coll = [sim.coll(b) for b in range(sim.B)]
        return dict(counts=_counts(sim), candidates=np.stack([c["candidates"] for c in coll]),
                    collisions=np.stack([c["coll"] for c in coll]),
                    density=np.stack([sim.density(b)[0] for b in range(sim.B)]))
    if kind == "argon":
        out = dict(counts=_counts(sim))
        if case["sampled"]:
            avg = [sim.avg(b) for b in range(sim.B)]
            out["mean_density"] = np.concatenate([a["density"].ravel() for a in avg])
            out["mean_phi"] = np.concatenate([a["phi"] for a in avg])
            out["mean_energy"] = np.concatenate([a["mean_energy"] for a in avg])
            if sim.B == 1:
                eepf, power = sim.eepf(), sim.power()
                out.update(eepf_bulk=eepf["bulk"], eepf_wall=eepf["wall"], power=power["power"], flux=power["flux"])
        if sim.B == 1 or not case["sampled"]:
            out["density"] = np.concatenate([sim.density(b).ravel() for b in range(sim.B)])
            out["phi"] = np.concatenate([sim.phi(b) for b in range(sim.B)])
        if sim.B == 1:
            wall, coll = sim.wall(), sim.coll()
            out.update(absorbed=wall["absorbed"], emitted=wall["see_emitted"], collisions=coll["coll"])
        return out
    out = dict(counts=_counts(sim), rho=sim.rho(), phi=sim.phi(), efield=sim.efield(), density=sim.density(),
               field_energy=sim.energy()[1])
    if kind == "langmuir":
        p = sim.get_particles(0)
        out.update({k: p[k].view(np.int32) if k == "id" else p[k] for k in ("cell", "off", "vx", "vy", "vz", "id")})
    elif case["renew"]:
        out["renewed"] = sim.renewed()
    return out


# ---- what a pass cannot do without ----------------------------------------------------
def work(case):
    """Bytes and operations of one pass.  A particle's step reads and writes
    its position (8 bytes) and the velocity components the fields change;
    a random draw reads its id (4 bytes), averages read every component, axial
    renewal reads and writes its displacement (8 bytes)."""
    kind = case["kind"]
    if kind == "poisson":
        nodes = case["cells"] + 1
        return dict(bytes=24.0 * nodes, flops=20.0 * nodes)
    if kind in ("train", "forward"):
        widths = _widths(case)
        params = sum((a + 1) * b for a, b in zip(widths[:-1], widths[1:]))
        io = 4.0 * case["batch"] * (widths[0] + widths[-1])
        if kind == "forward":
            return dict(bytes=io + 2.0 * params, flops=2.0 * case["batch"] * params)
        return dict(bytes=case["steps"] * (io + 24.0 * params), flops=6.0 * case["steps"] * case["batch"] * params)
    if kind == "langmuir":
        n, per, ops = case["n"], 24, 30
    elif kind == "box":
        n, per, ops = 2 * case["n"], 32 + (16 if case["renew"] else 0), 50
    elif kind == "argon":
        n, per, ops = case["total"], 36 if case["sampled"] else 28, 120
    else:
        n, per, ops = len(EN_TD) * case["replicas"] * case["n"], 28, 120
    return dict(bytes=float(n) * per * case["steps"], flops=float(n) * ops * case["steps"])


# ---- the same results in 64 bits -------------------------------------------------------
def _exact_poisson(case, seed):
    cfg = _gap_config(case)
    rho = _charge_density(case, seed).astype(np.longdouble)
    n = case["cells"]
    dx = np.longdouble(cfg["length"]) / n
    if not case["bounded"]:
        rho = rho - rho.mean()
    g = rho * dx * dx / np.longdouble(cfg["eps0"])
    g[0] = 0.0
    slope = np.cumsum(g)                                      # G[i] = g[1] + ... + g[i]
    k = np.concatenate([[np.longdouble(0.0)], np.cumsum(slope)])  # K[i] = G[0] + ... + G[i-1]
    i = np.arange(len(rho))
    if case["bounded"]:
        phi0 = np.longdouble(cfg["v_amp"] * math.sin(2.0 * math.pi * cfg["v_freq"] * 1e-9 + cfg["v_phase"]))
        phi = phi0 + i * (k[n] - phi0) / n - k[:n + 1]
        ef = np.zeros(n + 1, np.longdouble)
        ef[1:-1] = (phi[:-2] - phi[2:]) / (2.0 * dx)
        half = dx / (2.0 * np.longdouble(cfg["eps0"]))
        ef[0] = (phi[0] - phi[1]) / dx - rho[0] * half
        ef[n] = (phi[n - 1] - phi[n]) / dx + rho[n] * half
    else:
        phi = i * (k[n] / n) - k[:n]
        phi = phi - phi.mean()
        ef = (np.roll(phi, 1) - np.roll(phi, -1)) / (2.0 * dx)
    return dict(phi=phi.astype(np.float64), efield=ef.astype(np.float64))


def _exact_box(case, seed):
    """The explicit leapfrog step on a periodic mesh in FP64 (torch)."""
    cfg = _box_config(case, seed)
    nc, dt, dx = cfg["n_cells"], cfg["dt"], cfg["length"] / cfg["n_cells"]
    parts = _box_particles(cfg, seed)
    pos = [p["cell"].double() + p["off"].double() for p in parts]
    vel = [list(p["v"].double()) for p in parts]

    def solve():
        dens = []
        for s, sp in enumerate(cfg["species"]):
            c = pos[s].long().clamp_(max=nc - 1)
            f = pos[s] - c
            left = torch.bincount(c, weights=1.0 - f, minlength=nc)
            right = torch.bincount(c, weights=f, minlength=nc)
            dens.append((left + torch.roll(right, 1)) * (sp["weight"] / dx))
        rho = sum(sp["charge"] * d for sp, d in zip(cfg["species"], dens)) + cfg["rho_bg"]
        g = (rho - rho.mean()) * (dx * dx / cfg["eps0"])
        g[0] = 0.0
        slope = torch.cumsum(g, 0)
        k = torch.cumsum(slope, 0)
        phi = torch.arange(nc, device=g.device) * (k[-1] / nc) - (k - slope)
        phi = phi - phi.mean()
        return dens, rho, phi, (torch.roll(phi, 1) - torch.roll(phi, -1)) / (2.0 * dx)

    dens, rho, phi, ef = solve()
    for _ in range(case["steps"]):
        for s, sp in enumerate(cfg["species"]):
            qm = sp["charge"] / sp["mass"]
            c = pos[s].long().clamp_(max=nc - 1)
            f = pos[s] - c
            e = [ef[c] * (1.0 - f) + ef[(c + 1) % nc] * f + cfg["e_ext"][0], cfg["e_ext"][1], cfg["e_ext"][2]]
            h = 0.5 * qm * dt
            t = [h * b for b in cfg["b_ext"]]
            r = [2.0 * a / (1.0 + sum(b * b for b in t)) for a in t]
            u = [vel[s][k] + h * e[k] for k in range(3)]
            p = [u[0] + u[1] * t[2] - u[2] * t[1], u[1] + u[2] * t[0] - u[0] * t[2], u[2] + u[0] * t[1] - u[1] * t[0]]
            u = [u[0] + p[1] * r[2] - p[2] * r[1], u[1] + p[2] * r[0] - p[0] * r[2], u[2] + p[0] * r[1] - p[1] * r[0]]
            vel[s] = [u[k] + h * e[k] for k in range(3)]
            pos[s] = torch.remainder(pos[s] + vel[s][0] * (dt / dx), nc)
        dens, rho, phi, ef = solve()
    out = dict(counts=None, rho=rho, phi=phi, efield=ef, density=torch.stack(dens),
               field_energy=float(0.5 * cfg["eps0"] * dx * (ef * ef).sum()))
    if case["kind"] == "langmuir":
        out.update(cell=None, off=None, vx=vel[0][0], vy=vel[0][1], vz=vel[0][2], id=None)
    return out


def _layers(widths, params):
    at, out = 0, []
    for a, b in zip(widths[:-1], widths[1:]):
        out.append(params[at:at + b * (a + 1)].reshape(b, a + 1))
        at += b * (a + 1)
    return out


def _predict(layers, x):
    h = x
    for i, w in enumerate(layers):
        h = h @ w[:, :-1].t() + w[:, -1]
        if i + 1 < len(layers):
            h = 0.5 * h * (1.0 + torch.erf(h * math.sqrt(0.5)))
    return h


def _exact_network(case, seed):
    widths = _widths(case)
    params = torch.from_numpy(_network_params(widths, seed)).double().cuda()
    x, t = (torch.from_numpy(a).double().cuda() for a in _network_batches(case, seed))
    b = case["batch"]
    if case["kind"] == "forward":
        return dict(y=_predict(_layers(widths, params), x[:b]))
    m, v, losses = torch.zeros_like(params), torch.zeros_like(params), []
    sets = len(x) // b
    for k in range(case["steps"]):
        params.requires_grad_(True)
        at = (k % sets) * b
        loss = ((_predict(_layers(widths, params), x[at:at + b]) - t[at:at + b]) ** 2).mean()
        g, = torch.autograd.grad(loss, params)
        losses.append(float(loss))
        m = 0.9 * m + 0.1 * g
        v = 0.999 * v + 0.001 * g * g
        mh, vh = m / (1.0 - 0.9 ** (k + 1)), v / (1.0 - 0.999 ** (k + 1))
        params = (params.detach() - 1e-3 * mh / (vh.sqrt() + 1e-8)).detach()
    return dict(losses=torch.tensor(losses, dtype=torch.float64), params=params)


def exact(case, seed):
    """Poisson, the boxes whose particles are made here and the network;
    collisions, births and renewals follow the library's own random draws."""
    kind = case["kind"]
    if kind == "poisson":
        return _exact_poisson(case, seed)
    if kind == "langmuir" or (kind == "box" and not case["renew"] and case["n"] <= HOST_LOADED):
        return _exact_box(case, seed)
    if kind in ("train", "forward"):
        return _exact_network(case, seed)
    return None
