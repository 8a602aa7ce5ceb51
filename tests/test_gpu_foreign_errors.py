"""An error that another call of the program has left with the HIP runtime is
not reported by the calls that only read."""
import ctypes as C

import numpy as np
import pytest

from gpu_helpers import small_argon

pytestmark = pytest.mark.gpu


def test_reads_after_a_failed_call_of_the_program():
    import paper_2609_17151_amd as P
    cfg, tabs = small_argon(n_init=2000)
    sim = P.Sim(cfg, tabs)
    sim.step(3)
    phi = sim.phi()
    # the runtime that the library and torch share
    hip = C.CDLL(next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line))

    def fail():
        assert hip.hipSetDevice(4096) != 0               # refused, and kept as the last error

    fail()
    sim.sync()
    fail()
    assert sim.counts()["step"] == 3
    fail()
    assert np.array_equal(sim.phi(), phi)
    fail()
    assert sim.windows() == []
    hip.hipGetLastError()                                # the error is the program's to clear
    sim.close()
