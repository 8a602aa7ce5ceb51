"""A sampled step's push samples every particle before its event, and the events
pass adds what the event changed: the sums are those of the particles as the
step leaves them, collided, renewed, born and untouched alike."""
import numpy as np
import pytest

import workloads as W
from gpu_helpers import small_argon

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pic():
    import paper_2609_17151_amd as P
    return P


def _sums(sim, cfg, s):
    """Flux density per node, its rounding scale, and the particles, from the state."""
    p = sim.get_particles(s)
    nc, dx, w = cfg["n_cells"], cfg["length"] / cfg["n_cells"], cfg["species"][s]["weight"]
    n = sim.n_nodes[0]
    c, f, v = p["cell"].astype(np.int64), p["off"].astype(np.float64), p["vx"].astype(np.float64)
    out = []
    for q in (v, np.abs(v)):
        g = np.bincount(c, (1 - f) * q, n) + np.bincount((c + 1) % n, f * q, n)
        g = g * w / dx
        if n == nc + 1:
            g[[0, -1]] *= 2.0
        out.append(g)
    return out[0], out[1], p


@pytest.mark.parametrize("schedule", [(4, 256, True), (4, 1024, False), (1, 256, False)])
@pytest.mark.parametrize("kind", ["argon", "renewal"])
def test_sums_are_those_of_the_particles_the_step_leaves(pic, kind, schedule):
    tabs = ()
    if kind == "argon":
        # half a per cent of the electrons collide in a step
        cfg, tabs = small_argon(n_init=6001)
    else:
        cfg = W.exb(n_per_species=9001, n_cells=96, length=0.00178)
        cfg["renew_lz"] = 5e-5                 # a transit of some ten electron steps
    sim = pic.Sim(cfg, tabs)
    sim.config_tiles(schedule[0], schedule[1], 0, 16)
    sim.config_events(schedule[2])
    sim.step(20)
    events = 0
    for _ in range(4):
        sim.reset_avg()
        sim.set_diag(True)
        c0 = sim.coll()["coll"].sum() if kind == "argon" else int(np.sum(sim.renewed()))
        sim.step(1)
        events += (sim.coll()["coll"].sum() if kind == "argon" else int(np.sum(sim.renewed()))) - c0
        flux = sim.power()["flux"]
        for s in range(2):
            want, scale, p = _sums(sim, cfg, s)
            # products of binary32 velocities and offsets (a few 2^-24) and the
            # fixed-point rounding of each particle's words
            assert np.all(np.abs(flux[s] - want) <= 1e-6 * scale.max()), (kind, s)
        # whole numbers: the bulk electrons' energies, in binary32 as sampled
        want, scale, p = _sums(sim, cfg, 0)
        e = sim.eepf()
        hme = np.float32(0.5 * cfg["species"][0]["mass"] / cfg["e_unit"])
        eps = hme * (p["vx"] * p["vx"] + p["vy"] * p["vy"] + p["vz"] * p["vz"])
        assert eps.dtype == np.float32
        nc = cfg["n_cells"]
        lo, hi = ((0, nc) if cfg["bc"] == 0 else
                  (int(np.floor(0.45 * nc)), int(np.ceil(0.55 * nc))))
        nb = e["bulk"].size
        b = (eps * np.float32(nb / 64.0)).astype(np.int64)[(p["cell"] >= lo) & (p["cell"] < hi)]
        assert np.array_equal(e["bulk"], np.bincount(b[b < nb], minlength=nb))
    assert events > 20
