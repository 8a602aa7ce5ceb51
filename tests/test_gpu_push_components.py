"""The push leaves out the velocity components its fields do not change, and
deposits with one packed word per particle: steps under every direction of the
imposed fields against the oracle, a batch that mixes them against its
discharges alone, and more particles in one cell than a packed word holds."""
import numpy as np
import pytest

import workloads as W
from gpu_helpers import compare_species, small_argon, to_oracle

pytestmark = pytest.mark.gpu

# imposed E (in units of a typical field) and B (in units of 0.02 T)
FIELDS = {
    "none": ((0, 0, 0), (0, 0, 0)),
    "e_y": ((0, 1, 0), (0, 0, 0)),
    "e_z": ((0, 0, 1), (0, 0, 0)),
    "b_x": ((0, 0, 0), (1, 0, 0)),
    "b_y": ((0, 0, 1), (0, 1, 0)),
    "b_z": ((0, 1, 0), (0, 0, 1)),
    "b_y_e_y": ((0, 1, 0), (0, 1, 0)),
    "oblique": ((1, 1, 1), (0.5, 0.7, 0.3)),
}


@pytest.fixture(scope="module")
def pic():
    import paper_2609_17151_amd as P
    return P


def _fields(cfg, name):
    e, b = FIELDS[name]
    cfg["e_ext"] = [2e4 * v for v in e]
    cfg["b_ext"] = [0.02 * v for v in b]
    return cfg


@pytest.mark.parametrize("name", list(FIELDS))
@pytest.mark.parametrize("sampled", [False, True])
def test_box_step_matches_oracle(pic, name, sampled):
    # a periodic box (no walls, no draws), one step from identical states:
    # binary32 rounding of the push, 1e-6 as for every single step
    cfg = _fields(W.exb(n_per_species=5003, n_cells=96), name)
    sim = pic.Sim(cfg)
    sim.set_diag(sampled)
    sim.step(3)
    o = to_oracle(sim, cfg)
    sim.step(1)
    o.step(1)
    for s in range(2):
        r = compare_species(sim.get_particles(s), o.get_particles(s), cfg, cfg["species"][s]["vth"])
        assert r["id_equal"] and r["cell_mismatch"] == 0, (name, s)
        assert r["max_dx_over_L"] < 1e-6 and r["max_rel_v"] < 1e-6, (name, s, r["max_rel_v"])


@pytest.mark.parametrize("name", list(FIELDS))
@pytest.mark.parametrize("sampled,fused", [(False, False), (False, True), (True, False)])
def test_argon_step_matches_oracle(pic, name, sampled, fused):
    # walls, collisions, births: ids exact, velocities (the components the
    # push does not carry reach the events from the particle's slot) to 1e-6
    # but for one decision on a rounding edge, the energy carried into the
    # walls to 1e-5 (binary32 energies and velocities) and 2^-20 eV for every
    # particle (fixed point)
    cfg, tabs = small_argon(n_init=6001)
    _fields(cfg, name)
    sim = pic.Sim(cfg, tabs)
    sim.config_tiles(4, 256, 0, 16)
    sim.config_events(fused)
    sim.set_diag(sampled)
    sim.step(20)
    o = to_oracle(sim, cfg, tabs)
    w0, a0 = sim.wall_energy(), sim.wall()["absorbed"].copy()
    sim.step(4)
    o.step(4)
    for s in range(2):
        pg, po = sim.get_particles(s), o.get_particles(s)
        assert np.array_equal(pg["id"], po["id"]), (name, s)
        r = compare_species(pg, po, cfg, cfg["species"][s]["vth"])
        assert np.sum((r["rel_v"] > 4e-6) | (r["dx"] > 4e-6 * cfg["length"])) <= 1, (name, s)
    c = o.counters()
    absorbed = sim.wall()["absorbed"] - a0
    assert np.array_equal(absorbed, c["absorbed"]) and absorbed.sum() > 0, name
    fixed = absorbed * 2.0 ** -20 * cfg["e_unit"] * cfg["species"][0]["weight"]
    assert np.all(np.abs(sim.wall_energy() - w0 - c["wall_energy"]) <= 1e-5 * c["wall_energy"] + fixed), name


def test_batch_of_mixed_fields_equals_single_runs(pic):
    # the launch carries every component any of its discharges needs; each
    # discharge alone carries its own: the same state, bit for bit
    cfgs = []
    for i, name in enumerate(("none", "b_y", "oblique")):
        cfg, tabs = small_argon(n_init=3000 + 17 * i, seed=30 + i)
        cfgs.append(_fields(cfg, name))
    both = pic.Sim(cfgs, tabs)
    both.step(40)
    for b, cfg in enumerate(cfgs):
        one = pic.Sim(cfg, tabs)
        one.step(40)
        for s in range(2):
            pa, pb = both.get_particles(s, b), one.get_particles(s)
            for k in ("cell", "off", "vx", "vy", "vz", "id"):
                assert np.array_equal(pa[k], pb[k]), (b, s, k)
        assert np.array_equal(both.rho(b), one.rho())
        assert np.array_equal(both.wall_energy(b), one.wall_energy())


@pytest.mark.parametrize("cells,at,bounded", [(2, 1, False), (3, 2, True)])
def test_more_particles_in_one_cell_than_a_packed_word_holds(pic, cells, at, bounded):
    # 2e7 resting particles in the last cell: every workgroup's run of tiles
    # passes 65,535 particles of that cell; the density is n (1 - f) and n f
    # on the cell's two nodes, exactly (f = 3/8 is exact in every format)
    n = 20_000_000
    sp = W.species(-1.0, 1.0, 1.0, 0, 1.0, capacity=n, load=W.LOAD_NONE)
    cfg = W.base_config(n_cells=cells, bc=1 if bounded else 0, field_solve=0, length=float(cells), dt=0.01, species=[sp])
    sim = pic.Sim(cfg)
    z = np.zeros(n, np.float32)
    sim.set_particles(0, np.full(n, at, np.int32), np.full(n, 0.375, np.float32), z, z, z,
                      np.arange(n, dtype=np.uint32), n, 0)
    expect = np.zeros(cells + (1 if bounded else 0))
    right = at + 1 if bounded else (at + 1) % cells
    expect[at] += 0.625 * n
    expect[right] += 0.375 * n * (2.0 if bounded and right == cells else 1.0)
    for ppt, thr in ((4, 1024), (4, 256), (1, 256)):
        sim.config_tiles(ppt, thr, 0)
        sim.step(1)
        assert np.array_equal(sim.density()[0], expect), (ppt, thr)


@pytest.mark.parametrize("ppt,thr,fused", [(4, 1024, False), (1, 256, True)])
def test_more_segments_than_a_wave_has_lanes(pic, ppt, thr, fused):
    # up to 64 segments a wave holds the tile table in its lanes, beyond that
    # it lies in LDS: discharges of a batch of 33 (66 segments, some retired)
    # equal single runs bit for bit
    cfgs, tabs = [], None
    for i in range(33):
        cfg, tabs = small_argon(n_init=300 + 97 * i, seed=60 + i, n_cells=40 + 3 * i)
        cfgs.append(cfg)
    both = pic.Sim(cfgs, tabs)
    both.config_tiles(ppt, thr, 0, 16)
    both.config_events(fused)
    both.set_diag(True)
    both.retire(4)
    both.step(24)
    for b in (0, 5, 31, 32):
        one = pic.Sim(cfgs[b], tabs)
        one.set_diag(True)
        one.step(24)
        for s in range(2):
            pa, pb = both.get_particles(s, b), one.get_particles(s)
            for k in ("cell", "off", "vx", "vy", "vz", "id"):
                assert np.array_equal(pa[k], pb[k]), (b, s, k)
        assert np.array_equal(both.coll(b)["coll"], one.coll()["coll"])
        assert np.array_equal(both.phi(b), one.phi())
        assert np.array_equal(both.avg(b)["mean_energy"], one.avg()["mean_energy"])
    assert both.counts(4)["step"] == 0


def test_three_species_match_oracle(pic):
    # a third species (heavier ions beside the first) in a batch of two
    # discharges: every segment takes its own constants
    cfgs = []
    for i in range(2):
        cfg = W.exb(n_per_species=2003 + i, n_cells=64, seed=70 + i)
        third = dict(cfg["species"][1], mass=2.0 * cfg["species"][1]["mass"], n_init=1001, capacity=1001)
        cfg["species"] = cfg["species"] + [third]
        cfgs.append(cfg)
    sim = pic.Sim(cfgs)
    sim.step(2)
    refs = [to_oracle(sim, cfg, batch=b) for b, cfg in enumerate(cfgs)]
    sim.step(1)
    for b, (cfg, o) in enumerate(zip(cfgs, refs)):
        o.step(1)
        for s in range(3):
            r = compare_species(sim.get_particles(s, b), o.get_particles(s), cfg, cfg["species"][s]["vth"])
            assert r["id_equal"] and r["cell_mismatch"] == 0, (b, s)
            assert r["max_dx_over_L"] < 1e-6 and r["max_rel_v"] < 1e-6, (b, s)
