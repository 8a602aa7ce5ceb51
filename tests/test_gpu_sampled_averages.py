"""The time averages of one sampled step against their definition, formed here in
FP64 from the step's own density, field, flux and momentum flux: meshes on both
sides of a node per thread (1024), one to four species, walls and none."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pic():
    import paper_2609_17151_amd as P
    return P


@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("species", [1, 2, 3, 4])
@pytest.mark.parametrize("cells", [3, 64, 400, 1022, 1023, 1024, 1025, 1300])
def test_terms_of_one_step(pic, cells, species, bc):
    base = W.exb(n_per_species=7001, n_cells=cells)
    sps = []
    for s in range(species):
        sp = dict(base["species"][min(s, 1)])
        if s > 1:
            sp["mass"] = sp["mass"] / (3.0 * s)
            sp["vth"] = sp["vth"] * 2.0
        sps.append(sp)
    cfg = dict(base, species=sps, bc=bc, b_ext=[0.0, 0.0, 0.0], e_ext=[1e3, 0.0, 0.0])
    sim = pic.Sim(cfg)
    sim.step(3)
    sim.set_diag(True)
    sim.step(1)                              # stores the flux of the step before
    g0 = sim.power()["flux"]
    sim.reset_avg()
    sim.step(1)
    pw, avg, dens, e, phi = sim.power(), sim.avg(), sim.density(), sim.efield(), sim.phi()
    assert pw["samples"] == 1.0 and avg["samples"] == 1.0
    assert np.array_equal(avg["density"], dens) and np.array_equal(avg["phi"], phi)
    n, dx, dt = dens.shape[1], cfg["length"] / cells, cfg["dt"]
    i = np.arange(n)
    if bc == 0:
        il, ir, h = (i - 1) % n, (i + 1) % n, 2 * dx
    else:
        il, ir = np.maximum(i - 1, 0), np.minimum(i + 1, n - 1)
        h = (ir - il) * dx
    for s in range(species):
        m, q = sps[s]["mass"], sps[s]["charge"]
        G, M, nd = pw["flux"][s], pw["momentum"][s], dens[s]
        ok = nd > 0
        u = np.where(ok, G / np.where(ok, nd, 1.0), 0.0)
        K = np.where(ok, m * G * G / np.where(ok, nd, 1.0), 0.0)
        P = m * M - K
        acc = m * (G - g0[s]) / dt
        dk, dp = (K[ir] - K[il]) / h, (P[ir] - P[il]) / h
        # the same FP64 operations but for the order of a few: 1e-12 of the
        # largest of the terms that are added
        for what, want, scale in (("power", q * G * (e + 1e3), np.abs(q * G * (e + 1e3))),
                                  ("inertia", u * (acc + dk), np.abs(u) * (np.abs(acc) + np.abs(K).max() / dx)),
                                  ("pressure", u * dp, np.abs(u) * np.abs(P).max() / dx)):
            assert np.all(np.abs(pw[what][s] - want) <= 1e-12 * scale.max()), (what, s)
