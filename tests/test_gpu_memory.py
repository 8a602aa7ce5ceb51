"""Device memory of a context per particle slot, and the storage of the step's
events in contexts that get their first collision table after a run."""
import ctypes as C

import numpy as np
import pytest
import torch

import workloads as W
from gpu_helpers import small_argon

pytestmark = pytest.mark.gpu

SMALL = 32 << 20         # what does not grow with the slots: sums and fields of up to 400 nodes, the windows' ring
TILES = 16.0 / 256       # two arrays of 4 bytes and one of 8 per 256 slots


@pytest.fixture(scope="module")
def pic():
    import paper_2609_17151_amd as P
    return P


def _held(make):
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    sim = make()
    return sim, torch.cuda.memory_allocated() - before


def _empty(cfg, capacity):
    return dict(cfg, species=[dict(sp, load=W.LOAD_NONE, n_init=0, capacity=capacity) for sp in cfg["species"]])


def test_a_box_without_events_holds_its_particles_only(pic):
    # two copies of six four-byte arrays
    slots = 2 * 16384 * 4096
    sim, held = _held(lambda: pic.Sim(_empty(W.exb(n_cells=64), slots // 2)))
    assert held <= (48 + TILES) * slots + SMALL
    sim.close()


@pytest.mark.parametrize("tiles", [8192, 8193])
def test_events_and_births_of_large_contexts(pic, tiles):
    # the particles' copies, 32 bytes of event records and a birth (36 bytes)
    # for every sixteenth slot; up to 2^26 slots (16384 tiles of 4096) one for
    # every fourth
    slots = 2 * tiles * 4096
    cfg, tabs = small_argon()
    sim, held = _held(lambda: pic.Sim(_empty(cfg, slots // 2), tabs))
    births = 36 / 4 if slots <= 1 << 26 else 36 / 16
    assert held <= (48 + 32 + births + TILES) * slots + SMALL
    sim.close()


def _run(sim, steps=40):
    sim.step(steps)
    sim.sync()
    parts = [sim.get_particles(s) for s in range(2)]
    return ([p[k] for p in parts for k in ("cell", "off", "vx", "vy", "vz", "id")] +
            [sim.phi(), sim.coll()["coll"], sim.wall()["absorbed"], np.array(sim.counts()["next_id"])])


def _capacity(cfg, capacity):
    return dict(cfg, species=[dict(sp, capacity=capacity) for sp in cfg["species"]])


@pytest.mark.parametrize("schedule", [None, (4, 256, True), (1, 256, True), (4, 256, False)])
def test_a_large_context_runs_as_a_small_one(pic, schedule):
    # the same discharge in a context that stages births for tiles of 4096,
    # until a schedule whose push does its own events is set (after some steps
    # replayed from a captured graph, with the old staging)
    n = 60_000
    cfg, tabs = small_argon(n_init=n, weight=6e13 / n)
    runs = []
    for capacity in (4 * n, (1 << 25) + 1):
        sim = pic.Sim(_capacity(cfg, capacity), tabs)
        sim.step(64)
        sim.sync()
        before = torch.cuda.memory_allocated()
        if schedule:
            sim.config_tiles(*schedule[:2], 0, 16)
            sim.config_events(schedule[2])
            sim.config_events(schedule[2])
        grown = torch.cuda.memory_allocated() - before
        slots = 2 * ((1 << 25) + 4096)
        more = int((36 / 4 - 36 / 16) * slots) if capacity > 4 * n and schedule and schedule[2] else 0
        assert abs(grown - more) <= 4096
        runs.append(_run(sim, 64))
        sim.close()
    for x, y in zip(*runs):
        assert np.array_equal(x, y)


def test_no_memory_for_the_denser_staging(pic):
    # the schedule is taken all the same, its events by the events kernel
    n = 60_000
    cfg, tabs = small_argon(n_init=n, weight=6e13 / n)
    full = []
    sim = pic.Sim(_capacity(cfg, (1 << 25) + 1), tabs)
    sim.close()
    real = torch.cuda.caching_allocator_alloc

    def refusing(size, *a):
        return None if full else real(size, *a)

    torch.cuda.caching_allocator_alloc = refusing
    try:
        sim = pic.Sim(_capacity(cfg, (1 << 25) + 1), tabs)
        full.append(1)
        sim.config_tiles(4, 256, 0, 16)
        sim.config_events(True)
        sim.profile(True)
        sim.step(2)
        assert sim.timing()["events_n"] == 2
        sim.profile(False)
        got = _run(sim)
        sim.close()
    finally:
        torch.cuda.caching_allocator_alloc = real
    small = pic.Sim(_capacity(cfg, 4 * n), tabs)
    small.config_tiles(4, 256, 0, 16)
    small.step(2)
    for x, y in zip(got, _run(small)):
        assert np.array_equal(x, y)
    small.close()


def test_collisions_from_a_later_step_on(pic):
    # a periodic box streams, then gets a collision table: from there on the
    # same as a box that had it all along but whose gas was collisionless until
    # then (its table's cross section is zero, so that no particle is a candidate)
    cfg = dict(W.maxwell_swarm(n_particles=5000, gas_mass=W.AR_MASS, dt=2e-11)[0], field_solve=0)
    e = np.logspace(-4, 4, 400)
    one = dict(species=0, kind=W.XS_ELASTIC, threshold=0.0, energy=e, sigma=np.full_like(e, 1e-19))
    late, early = pic.Sim(cfg), pic.Sim(cfg)
    early.load_xsec(0, W.XS_ELASTIC, 0.0, e, np.full_like(e, 1e-40))
    for sim in (late, early):
        sim.step(7)
    assert early.coll()["candidates"][0] == 0
    a, b = late.get_particles(0), early.get_particles(0)
    for k in ("cell", "off", "vx", "vy", "vz", "id"):
        assert np.array_equal(a[k], b[k]), k
    late.load_xsec(one["species"], one["kind"], one["threshold"], one["energy"], one["sigma"])
    late.step(40)
    late.sync()
    c = late.coll()
    assert c["candidates"][0] > 0 and c["coll"][0][0] > 0
    assert c["candidates"][0] == c["nulls"][0] + c["coll"][0].sum()
    # a table that is there from the start gives the candidates of the id draws
    other = pic.Sim(cfg, [one])
    assert other.numax(0) == late.numax(0)


def test_a_network_of_the_chain_holds_no_rows_for_other_kernels(pic):
    # per sample: every layer's input with its ones and output gradient in BF16
    # (rows of 32 and 16), the hidden layers' pre-activations in FP32
    widths, batch = (5, 64, 64, 48), 65536
    pairs = list(zip(widths[:-1], widths[1:]))
    row = sum(2 * ((a + 32) // 32 * 32 + (b + 15) // 16 * 16) for a, b in pairs) + 4 * sum(widths[1:-1])
    lib, h, asked = pic.load_library(), C.c_void_p(), []

    def alloc(n, user):
        asked.append(n)
        return torch.cuda.caching_allocator_alloc(int(n))

    hooks = pic.ALLOC_FN(alloc), pic.FREE_FN(lambda p, user: torch.cuda.caching_allocator_delete(p))
    a = pic.PicAllocator(*hooks, None)
    w = (C.c_int32 * len(widths))(*widths)
    assert lib.pic_mlp_create(w, len(widths), batch, C.byref(a), None, C.byref(h)) == pic.OK
    assert sum(asked) <= row * batch + (4 << 20)
    lib.pic_mlp_free(h)
