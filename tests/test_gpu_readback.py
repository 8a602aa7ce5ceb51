"""Readback of device state through the context's pinned buffer: every selector
on the largest context shape, sizes and selectors that are refused, the field
solve with and without a density, and two threads with a context each."""
import ctypes as C
import threading

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pic():
    import paper_2609_17151_amd as P
    return P


def _largest(n=600):
    cfg = W.exb(n_per_species=n, n_cells=4096)
    ion = cfg["species"][1]
    cfg["species"] = cfg["species"] + [dict(ion, mass=2.0 * ion["mass"]), dict(ion, mass=3.0 * ion["mass"])]
    return cfg


def test_every_selector_of_the_largest_shape(pic):
    # four species, 4096 cells, two discharges: the power sums and the wall
    # distributions are the largest readbacks (a mesh this large is not
    # sampled, so they read zero)
    sim = pic.Sim([_largest(), _largest(700)])
    sim.step(4)
    for b in range(2):
        n = 600 if b == 0 else 700
        assert sim.counts(b)["count"] == [n] * 4 and sim.counts(b)["step"] == 4
        assert sim.power(b)["flux"].shape == (4, 4096) and not np.any(sim.power(b)["flux"])
        assert sim.wall_edf(b)["counts"].shape == (4, 2, 256) and sim.avg(b)["samples"] == 0
        assert sim.wall_energy(b).shape == (4, 2) and sim.renewed(b).shape == (4,)
        assert sim.eepf(b)["bulk"].sum() == 0 and sim.coll(b)["candidates"].shape == (4,)
        # the integral of every species' density is its particles
        cfg = sim.cfgs[b]
        dx = cfg["length"] / 4096
        for s, sp in enumerate(cfg["species"]):
            np.testing.assert_allclose(sim.density(b)[s].sum() * dx, n * sp["weight"], rtol=1e-12)
        q, qp = sim.charge(b)
        assert abs(q - qp) <= 1e-12 * n * cfg["species"][0]["weight"] * W.E_CHARGE


def test_sampled_selectors_and_windows(pic):
    cfg = W.exb(n_per_species=3001, n_cells=1500)
    sim = pic.Sim([cfg, dict(cfg, seed=9)])
    sim.set_diag(True)
    sim.set_windows(1, 2)
    sim.step(4)
    w = sim.windows(1)
    assert len(w) == 2 and all(x["samples"] == 2 for x in w) and sim.avg(0)["samples"] == 4
    assert np.any(sim.power(0)["flux"]) and sim.eepf(1)["bulk"].sum() > 0
    assert np.isfinite(sim.power(1)["power"]).all()


def test_refused_sizes_and_selectors(pic):
    sim = pic.Sim(_largest())
    L = pic.load_library()
    buf = np.zeros(4096 * 32)
    p = buf.ctypes.data_as(C.c_void_p)
    need = {0: 8 * 12, 1: 8 * 4096, 4: 8 * 4 * 4096, 10: 8 * (1 + 6 * 4096), 15: 8 * (1 + 20 * 4096), 17: 8 * (4 * 512 + 5)}
    for what, size in need.items():
        assert L.pic_diag(sim.h, 0, what, p, size) == pic.OK, what
        assert L.pic_diag(sim.h, 0, what, p, size - 1) == pic.EINVAL, what
        assert L.pic_diag(sim.h, 0, what, None, size) == pic.EINVAL, what
    assert L.pic_diag(sim.h, 0, 99, p, buf.nbytes) == pic.EINVAL
    assert L.pic_diag(sim.h, 1, 0, p, buf.nbytes) == pic.EINVAL


def test_field_solve_with_and_without_a_density(pic):
    cfg = W.exb(n_per_species=5000, n_cells=500)
    sim = pic.Sim(cfg)
    sim.step(3)
    phi, ef = sim.poisson(0.0)                       # the last deposited density
    assert np.array_equal(phi, sim.phi()) and np.array_equal(ef, sim.efield())
    phi2, ef2 = sim.poisson(0.0, sim.rho())          # the same, handed over
    assert np.array_equal(phi2, phi) and np.array_equal(ef2, ef)


def test_two_threads_with_a_context_each(pic):
    import torch
    expect = {}
    for seed in (1, 2):
        one = pic.Sim(W.langmuir(n_particles=4000 + seed, seed=seed))
        one.step(40)
        expect[seed] = (one.phi(), one.counts())
    got = {}

    def work(seed):
        sim = pic.Sim(W.langmuir(n_particles=4000 + seed, seed=seed), stream=torch.cuda.Stream())
        for _ in range(40):
            sim.step(1)
            phi, counts = sim.phi(), sim.counts()
        got[seed] = (phi, counts)
        sim.close()

    threads = [threading.Thread(target=work, args=(s,)) for s in expect]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for seed, (phi, counts) in expect.items():
        assert np.array_equal(got[seed][0], phi) and got[seed][1] == counts
