"""Streaming steps after the first of a run solve for their field inside the
push, from sets of deposit sums that go round: a run of many steps gives the
same bits as its steps one by one, where each is finished by the finalize
kernel."""
import numpy as np
import pytest

import workloads as W

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
        out += [sim.phi(b), sim.efield(b), sim.density(b)]
    return out


def _same(a, b):
    assert len(a) == len(b)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


# both sides of a wave's 64 lanes x 4 nodes, of the waves, and of the largest
# mesh the push solves (1024 nodes)
@pytest.mark.parametrize("cells", [2, 3, 63, 64, 65, 255, 256, 257, 700, 1023, 1024, 1025])
@pytest.mark.parametrize("ppt,threads", [(1, 256), (4, 256), (4, 1024)])
def test_a_run_gives_the_bits_of_its_steps(pic, cells, ppt, threads):
    cfg = W.exb(n_per_species=6007, n_cells=cells)
    runs = []
    for parts in ([7], [1] * 7, [2, 3, 2], [4, 1, 2]):
        sim = pic.Sim(cfg)
        sim.config_tiles(ppt, threads, 0, 16)
        for n in parts:
            sim.step(n)
        runs.append(_state(sim))
        sim.close()
    for r in runs[1:]:
        _same(runs[0], r)


@pytest.mark.parametrize("sort", [0, 3])
def test_batches_of_meshes_replays_and_sampled_steps(pic, sort):
    # discharges of different meshes in one launch (a workgroup's tiles can
    # span several of them), one with its field switched off; captured chunks
    # replayed with reads and sampled steps between them
    cfgs = [W.exb(n_per_species=n, n_cells=c) for n, c in ((501, 64), (9001, 1000), (37, 5), (4096, 256))]
    cfgs[3]["field_solve"] = 0
    runs = []
    for one_by_one in (False, True):
        sim = pic.Sim(cfgs)
        sim.config_tiles(4, 256, sort, 16)
        out = []
        for n, sampled in ((97, False), (3, True), (64, False), (64, False), (2, False)):
            sim.set_diag(sampled)
            for k in ([1] * n if one_by_one else [n]):
                sim.step(k)
            out += _state(sim)
        runs.append(out)
        sim.close()
    _same(*runs)
