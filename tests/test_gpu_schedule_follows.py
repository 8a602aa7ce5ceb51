"""The schedule the library takes when none is set follows the particles the
host last saw: the number of events launches tells small tiles (none: the push
does its own events) from large ones (one per step)."""
import numpy as np
import pytest

import workloads as W
from gpu_helpers import small_argon

pytestmark = pytest.mark.gpu

LINE = 6_000_000


@pytest.fixture(scope="module")
def pic():
    import paper_2609_17151_amd as P
    return P


def _events_launches(sim, steps=2):
    sim.profile(True)
    sim.step(steps)
    n = sim.timing()["events_n"]
    sim.profile(False)
    return n


@pytest.mark.parametrize("n,large", [(1000, False), (LINE, False), (LINE + 1, True)])
def test_both_sides_of_the_line(pic, n, large):
    cfg, tabs = small_argon(n_init=n // 2, weight=6e13 / n)
    for s, sp in enumerate(cfg["species"]):
        sp["capacity"] = n
        sp["n_init"] = n // 2 + (n % 2 if s == 0 else 0)
    sim = pic.Sim(cfg, tabs)
    assert _events_launches(sim) == (2 if large else 0)
    sim.config_tiles(4, 1024, 0, 16)                     # an explicit schedule is taken as given
    assert _events_launches(sim) == 2
    sim.config_tiles(4, 256, 0, 16)
    sim.config_events(True)
    assert _events_launches(sim) == 0
    sim.close()


@pytest.mark.parametrize("batch,n,large", [(1, 2_000_000, False), (1, 2_000_002, True), (2, 2_000_004, False)])
def test_sampled_steps_of_one_discharge(pic, batch, n, large):
    cfg, tabs = small_argon(n_init=n // 2 // batch, weight=6e13 / n)
    for sp in cfg["species"]:
        sp["capacity"] = n
    sim = pic.Sim([cfg] * batch, tabs)
    assert _events_launches(sim) == 0                    # unsampled: far below the line
    sim.set_diag(True)
    assert _events_launches(sim) == (2 if large else 0)
    sim.set_diag(False)
    assert _events_launches(sim) == 0
    sim.close()


def _ionizing(pic, n, hot):
    # `hot` of n electrons at 20 eV, every one a candidate that ionizes with
    # probability 1 / 1.05 (a constant collision frequency far above 1 / dt);
    # the others, and all of them afterwards, are below the threshold
    cfg, tabs = W.maxwell_swarm(nu0=1e12, n_particles=n, te_ev=0.1, gas_mass=W.AR_MASS, kind=W.XS_IONIZATION)
    cfg["species"][0].update(capacity=2 * n, load=W.LOAD_NONE, n_init=0)
    sim = pic.Sim(cfg, [dict(tabs[0], threshold=15.8)])
    v = np.full(n, 1e5, np.float32)
    v[::n // hot] = 2.65e6
    z = np.zeros(n, np.float32)
    sim.set_particles(0, (np.arange(n) % cfg["n_cells"]).astype(np.int32), np.full(n, 0.5, np.float32), v, z, z,
                      np.arange(n, dtype=np.uint32), n, 0)
    return sim


@pytest.mark.parametrize("read", ["sync", "counts", "particles"])
def test_a_run_that_grows_takes_large_tiles(pic, read):
    sim = _ionizing(pic, 5_900_000, 236_000)
    assert _events_launches(sim, 1) == 0
    assert sim.counts()["count"][0] > LINE if read == "counts" else True
    if read == "sync":
        sim.sync()
    elif read == "particles":
        assert len(sim.get_particles(0)["id"]) > LINE
    assert _events_launches(sim, 1) == 1
    # thinned below the line it stays with large tiles, at half the line not
    for keep, launches in ((4_000_000, 1), (2_000_000, 0), (2_000_000, 0)):
        sim.thin(0, keep, keep)
        sim.sync()
        assert _events_launches(sim, 1) == launches, keep
    sim.close()


def test_particles_set_anew_are_judged_anew(pic):
    sim = _ionizing(pic, LINE + 500_000, 10)
    assert _events_launches(sim, 1) == 1
    p = sim.get_particles(0)
    n = LINE - 100_000
    sim.set_particles(0, *(p[k][:n] for k in ("cell", "off", "vx", "vy", "vz", "id")), p["next_id"], 1)
    assert _events_launches(sim, 1) == 0
    sim.close()


def test_retired_discharges_do_not_count(pic):
    n = 1_600_000
    cfg, tabs = small_argon(n_init=n, weight=6e13 / n)
    for sp in cfg["species"]:
        sp["capacity"] = 2 * n
    sim = pic.Sim([cfg, cfg], tabs)                      # 6.4e6 in all
    assert _events_launches(sim) == 2
    sim.retire(1)
    sim.sync(check=False)
    assert _events_launches(sim) == 2                    # 3.2e6: above half the line
    cfgs = [dict(cfg, species=[dict(sp, n_init=n // 2) for sp in cfg["species"]]) for _ in range(4)]
    sim.close()
    sim = pic.Sim(cfgs, tabs)
    assert _events_launches(sim) == 2
    for b in (1, 2, 3):
        sim.retire(b)
    assert _events_launches(sim) == 0
    sim.retire(1, False)
    sim.retire(2, False)
    sim.retire(3, False)
    assert _events_launches(sim) == 2
    sim.close()
