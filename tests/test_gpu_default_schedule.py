"""The schedule the library takes when none is set: the same run, bit for bit,
as with explicit ones, on both sides of its rule; and births as dense as a
larger tile stages."""
import numpy as np
import pytest

import workloads as W
from gpu_helpers import small_argon

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pic():
    import paper_2609_17151_amd as P
    return P


def _state(sim):
    out = []
    for b in range(sim.B):
        for s in range(sim.S):
            p = sim.get_particles(s, b)
            out += [p[k] for k in ("cell", "off", "vx", "vy", "vz", "id")]
        out += [sim.phi(b), sim.coll(b)["coll"], sim.wall()["absorbed"]]
    return out


@pytest.mark.parametrize("n", [700, 60_000, 4_100_000])
def test_default_schedule_gives_the_same_run(pic, n):
    # 4.1e6 per species is past the rule's 6e6 particles
    cfg, tabs = small_argon(n_init=n, weight=6e13 / n)
    for sp in cfg["species"]:
        sp["capacity"] = n + n // 8 + 4096
    runs = []
    for schedule in (None, (4, 1024, False), (4, 256, True)):
        sim = pic.Sim(cfg, tabs)
        if schedule:
            sim.config_tiles(schedule[0], schedule[1], 0, 16)
            sim.config_events(schedule[2])
        sim.step(20)
        runs.append(_state(sim))
        sim.close()
    for other in runs[1:]:
        for x, y in zip(runs[0], other):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("ppt,thr", [(4, 1024), (4, 512), (4, 256), (None, None)])
def test_the_default_stages_births_as_dense_as_large_tiles(pic, ppt, thr):
    # 240 electrons in a row ionize in one step (a cross section so large that
    # every one is a candidate and collides, energies far above threshold), the
    # other 3856 are below it: tiles of 1024 particles, the default's, drop no
    # birth that tiles of 4096 stage
    n, hot = 4096, 240
    cfg, tabs = W.maxwell_swarm(n_particles=n, nu0=1e9, dt=2e-11, te_ev=0.1, gas_mass=W.AR_MASS)
    e = np.logspace(-4, 4, 2000)
    sigma = np.full_like(e, 1e-17)
    cfg["species"][0]["capacity"] = 4 * n
    cfg["species"][0]["load"] = W.LOAD_NONE
    cfg["species"][0]["n_init"] = 0
    cfg["gas_density"] = 1e26
    sim = pic.Sim(cfg, [dict(species=0, kind=W.XS_IONIZATION, threshold=15.8, energy=e, sigma=sigma)])
    if ppt:
        sim.config_tiles(ppt, thr, 0, 16)
        sim.config_events(thr == 256)
    v = np.full(n, 1e5, np.float32)
    v[:hot] = 1.3e8                                    # about 48 keV
    z = np.zeros(n, np.float32)
    cell = (np.arange(n) % cfg["n_cells"]).astype(np.int32)
    sim.set_particles(0, cell, np.full(n, 0.5, np.float32), v, z, z, np.arange(n, dtype=np.uint32), n, 0)
    sim.step(1)
    sim.sync()
    c = sim.counts()
    born = c["count"][0] - n
    assert c["flags"] == 0 and born == sim.coll()["coll"][0][0] and born == c["next_id"][0] - n
    assert born > 0.5 * hot
