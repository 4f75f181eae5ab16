"""Waits of launches that hold whole sweeps (small lattices): one that passes its
limit, set low from the host, ends the launch normally and the call reports it,
whichever wave of a block gives up."""
import numpy as np
import pytest

import paper_0904_0642_amd as su3hb

pytestmark = pytest.mark.gpu


def test_limit_is_checked():
    g = su3hb.Lattice([4, 4], seed=1)
    for bad in (0, (1 << 24) + 1):
        with pytest.raises(su3hb.SU3HBError) as ei:
            su3hb.su3hb_set_wait_limit(g.handle, bad)
        assert ei.value.code == su3hb.EINVAL


@pytest.mark.parametrize("ext,nlat,mask,prec", [([32, 32], 1, 0, su3hb.FP64_18), ([32, 64], 1, 0, su3hb.FP32_12),
                                                ([4, 4, 4, 4], 1, 0, su3hb.FP64_18),
                                                ([6, 4, 4, 4], 2, 0b0111, su3hb.FP32_18)])
def test_a_wait_past_its_limit_is_reported(ext, nlat, mask, prec):
    # a slice takes some 4 us, a poll about 0.5 us: one poll is too few for
    # blocks that wait for each other 160 times and more
    kw = dict(nlat=nlat, dlt_mask=mask, precision=prec, seed=6)
    for call in (lambda g: g.sweep_measure(5.7, n_sweeps=40), lambda g: g.sweep(5.7, n_sweeps=40, stats=True)):
        g = su3hb.Lattice(ext, **kw)
        su3hb.su3hb_set_wait_limit(g.handle, 1)
        with pytest.raises(su3hb.SU3HBError) as ei:
            call(g)
        assert ei.value.code == su3hb.EHIP and "limit" in str(ei.value)
    # the longest limit changes nothing
    a, b = (su3hb.Lattice(ext, **kw) for _ in range(2))
    su3hb.su3hb_set_wait_limit(b.handle, 1 << 24)
    assert np.array_equal(a.sweep_measure(5.7, n_sweeps=5), b.sweep_measure(5.7, n_sweeps=5), equal_nan=True)
    assert np.array_equal(a.get_links(), b.get_links())
