"""get_links and set_links at the sizes where they change from the runtime's own
copy to a ring of pinned slots, up to pieces, parts and the staging buffer
that end anywhere: the bytes that went in come back, and a lattice that was
refused keeps its links."""
import numpy as np
import pytest

import paper_0904_0642_amd as su3hb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ext", [
    [8, 8, 8, 14], [8, 8, 8, 16],           # 4.13 MB and 4.72 MB: below and above the line from the device
    [16, 14, 16, 16], [14, 14, 12, 26],     # 33.0 MB and 35.2 MB: below and above the line to the device
    [16, 16, 16, 16], [30, 26, 22, 30],     # 37.7 MB; 297 MB: more than the staging buffer
    [2, 131072], [6, 6, 6, 6, 6, 12],       # 75.5 MB of one row; six dimensions
])
def test_links_return_as_they_went(ext):
    a = su3hb.Lattice(ext, seed=3)
    want = a.get_links()
    b = su3hb.Lattice(ext, start=su3hb.COLD, seed=4)
    b.set_links(want)
    assert np.array_equal(b.get_links(), want)
    # the last matrix of the input is not in SU(3): nothing is written
    bad = want.copy()
    bad.reshape(-1, 3, 3)[-1] *= 1.5
    with pytest.raises(su3hb.SU3HBError) as ei:
        b.set_links(bad)
    assert ei.value.code == su3hb.ENOTSU3
    assert np.array_equal(b.get_links(), want)


def test_pinned_memory_and_a_stream_of_its_own():
    import torch
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        a = su3hb.Lattice([16, 16, 16, 16], seed=3)
        a.sweep(5.5)
        want = a.get_links()
        pinned = torch.empty(want.shape, dtype=torch.complex128, pin_memory=True).numpy()
        pinned[:] = want
        b = su3hb.Lattice([16, 16, 16, 16], seed=8)
        b.sweep(5.5)
        b.set_links(pinned)
        assert np.array_equal(b.get_links(), want)
