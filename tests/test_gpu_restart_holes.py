"""A field solved anew between steps while absorbed particles still leave holes:
the same field as after a compaction, and no flag."""
import numpy as np
import pytest

import workloads as W
from gpu_helpers import small_argon

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pic():
    import paper_2609_17151_amd as P
    return P


def _run(pic, cfg, tabs, compact_every):
    sim = pic.Sim(cfg, tabs)
    sim.config_tiles(4, 256, 0, compact_every)
    sim.step(15)
    assert sum(sim.wall()["absorbed"].ravel()) > 0
    return sim


def test_particles_of_one_species_replaced(pic):
    cfg, tabs = small_argon(n_init=30000)
    out = []
    for every in (1, 64):                    # 64: the first species keeps its holes
        sim = _run(pic, cfg, tabs, every)
        n = 29000
        cell = (np.arange(n) % cfg["n_cells"]).astype(np.int32)
        v = np.zeros(n, np.float32)
        sim.set_particles(1, cell, np.full(n, 0.25, np.float32), v, v, v, np.arange(n, dtype=np.uint32), n, 15)
        sim.sync()
        out.append((sim.density(), sim.phi()))
    for a, b in zip(*out):
        assert np.array_equal(a, b)


def test_charge_of_the_electrode_replaced(pic):
    cfg, tabs = small_argon(n_init=30000)
    cfg = dict(cfg, drive=1, cap=1e-9)
    out = []
    for every in (1, 64):
        sim = _run(pic, cfg, tabs, every)
        sim.set_circuit(1e-7)
        sim.sync()
        out.append((sim.density(), sim.phi()))
    for a, b in zip(*out):
        assert np.array_equal(a, b)
