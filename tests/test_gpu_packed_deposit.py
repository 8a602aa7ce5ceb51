"""The packed deposit word counts at most 65,535 particles of a cell; a
workgroup whose run of tiles is longer flushes its histogram in between.  Every
shape and kind of step is run on so many particles that every workgroup's run
is longer, however many workgroups the GPU holds, with a run's particles in one
or two neighbouring cells; the densities equal, bit for bit, those of the
deposit that a start or restart uses, which adds each particle's two weights."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

PACKED = 65_535
CELLS = 96


@pytest.fixture(scope="module")
def pic():
    import paper_2609_17151_amd as P
    return P


def _particles():
    # workgroups of 256 threads: at most eight on a compute unit (32 waves of
    # 64 lanes); larger ones are fewer.  With 1.05 times that many runs of
    # 65,535 particles every workgroup passes the limit.
    wg = 8 * torch.cuda.get_device_properties(0).multi_processor_count
    n = int(1.05 * wg * (PACKED + 4096))
    assert n / wg > PACKED
    # and a cell holds several runs: a run's particles share a cell or two, so
    # that without the flush its word would overflow
    assert n / CELLS > 2 * PACKED
    return n


def _sim(pic, kind):
    # the first species in order of position, cold; a second one of a few
    # particles, whose replacement by itself makes the library deposit anew
    n = _particles()
    few = W.species(1.0, 1.0, 1.0, 1000, 1.0, capacity=4096, load=W.LOAD_RANDOM)
    many = W.species(-1.0, 1.0, 1.0, n, 1.0, capacity=n + (1 << 20), load=W.LOAD_STRATIFIED)
    cfg = W.base_config(n_cells=CELLS, bc=1 if kind == "bounded" else 0, field_solve=1, length=float(CELLS),
                        dt=0.01, eps0=1e12, rho_bg=0.0, species=[many, few])
    if kind == "renewing":
        cfg["renew_lz"] = 50.0
    return pic.Sim(cfg)


def _check(sim, what):
    sim.sync()
    got = sim.density()
    p = sim.get_particles(1)
    step = sim.counts()["step"]
    sim.set_particles(1, p["cell"], p["off"], p["vx"], p["vy"], p["vz"], p["id"], p["next_id"], step)
    again = sim.density()
    assert np.array_equal(got, again), what
    assert got[0].sum() > 0


STREAMING = ((4, 1024), (4, 512), (8, 256), (4, 256), (2, 256), (1, 256))
GENERAL = ((4, 1024, 0), (4, 512, 0), (8, 512, 0), (8, 256, 0), (4, 256, 0), (2, 256, 0), (1, 256, 0),
           (4, 256, 1), (2, 256, 1), (1, 256, 1))


def test_streaming_steps(pic):
    # one step (its field from the last finalize) and three, of which two solve
    # for their field themselves; then sampled steps
    sim = _sim(pic, "streaming")
    for ppt, thr in STREAMING:
        sim.config_tiles(ppt, thr, 0, 1)
        for steps in (1, 3):
            sim.step(steps)
            _check(sim, (ppt, thr, steps))
    sim.set_diag(True)
    for ppt, thr in STREAMING:
        sim.config_tiles(ppt, thr, 0, 1)
        sim.step(1)
        _check(sim, (ppt, thr, "sampled"))
    sim.close()


@pytest.mark.parametrize("kind", ["renewing", "bounded"])
def test_general_steps(pic, kind):
    sim = _sim(pic, kind)
    for sampled in (False, True):
        sim.set_diag(sampled)
        for ppt, thr, fused in GENERAL:
            sim.config_tiles(ppt, thr, 0, 1)                # absorbed particles are compacted away at once
            sim.config_events(fused)
            sim.step(1)
            _check(sim, (ppt, thr, fused, sampled))
    sim.close()
