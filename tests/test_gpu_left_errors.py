"""An error that another HIP call of the thread has left behind is not the sweeps':
they run, and say so, in every form of a slice."""
import ctypes as C

import numpy as np
import pytest

import paper_0904_0642_amd as su3hb

pytestmark = pytest.mark.gpu


@pytest.fixture
def hip():
    import torch
    torch.cuda.synchronize()
    lib = C.CDLL(next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line))
    yield lib
    lib.hipGetLastError()  # torch's next call would report it


def leave_an_error(hip):
    assert hip.hipSetDevice(C.c_int(12345)) != 0


@pytest.mark.parametrize("ext", [[4, 4, 4, 4], [8, 8, 8, 8], [16, 16, 16, 16], [24, 24, 24, 12]])
def test_sweeps_run(ext, hip):
    # whole sweeps in one launch, lanes and waves, planes on waves, a thread per link
    a, b = (su3hb.Lattice(ext, precision=su3hb.FP32_18, seed=3) for _ in range(2))
    for g in (a, b):
        g.sweep(5.7)
    want = [b.sweep_measure(5.7, n_sweeps=2)]
    b.overrelax(5.7)
    leave_an_error(hip)
    got = [a.sweep_measure(5.7, n_sweeps=2)]
    leave_an_error(hip)
    a.overrelax(5.7)
    assert np.array_equal(got[0], want[0], equal_nan=True)
    leave_an_error(hip)
    assert np.array_equal(a.plaquette(5.7), b.plaquette(5.7), equal_nan=True)
    assert np.array_equal(a.get_links(), b.get_links()) and a.get_state() == b.get_state()
