"""The compaction with and without its scan pass (few tiles in the context, or
many): the same run, bit for bit, and the particles in their order."""
import numpy as np
import pytest

import workloads as W
from gpu_helpers import small_argon

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pic():
    import paper_2609_17151_amd as P
    return P


@pytest.mark.parametrize("every", [1, 4])
@pytest.mark.parametrize("n", [1, 255, 1023, 1024, 1025, 4097, 60_000])
def test_few_and_many_tiles_give_the_same_run(pic, n, every):
    # capacities of 2 x 2^18 and 2 x 4.5e6 slots: 512 and 8790 tiles of 1024
    runs = []
    for cap in (1 << 18, 4_500_000):
        cfg, tabs = small_argon(n_init=n, weight=6e13 / max(n, 1000))
        for sp in cfg["species"]:
            sp["capacity"] = cap
        sim = pic.Sim(cfg, tabs)
        sim.config_tiles(4, 256, 0, every)
        sim.config_events(True)
        # a third of the particles start next to a wall on their way out
        for s in range(2):
            p = sim.get_particles(s)
            m = np.arange(n) % 3 == 0
            p["cell"][m] = 0
            p["vx"][m] = -np.abs(p["vx"][m]) - 1e5
            sim.set_particles(s, p["cell"], p["off"], p["vx"], p["vy"], p["vz"], p["id"], p["next_id"], 0)
        out = []
        for k in (1, 3, 8):
            sim.step(k)
            for s in range(2):
                p = sim.get_particles(s)
                out += [p[q] for q in ("cell", "off", "vx", "vy", "vz", "id")]
                # no births out of order: ids ascend within the survivors
                assert np.all(np.diff(p["id"].astype(np.int64)) > 0) and np.all(p["cell"] >= 0)
            c = sim.counts()
            assert c["flags"] == 0
            out += [np.asarray(c["count"]), sim.wall()["absorbed"]]
        runs.append(out)
        sim.close()
    assert runs[0][-1].sum() > 0 or n < 255
    for x, y in zip(*runs):
        assert np.array_equal(x, y)
