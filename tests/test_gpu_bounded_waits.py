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


def test_set_links_ends_the_error():
    g, ref = (su3hb.Lattice([4, 4, 4, 4], seed=9) for _ in range(2))
    ref.sweep(5.7, n_sweeps=2)
    links = ref.get_links()
    su3hb.su3hb_set_wait_limit(g.handle, 1)
    g.sweep(5.7, n_sweeps=40)
    for call in (lambda: g.plaquette(5.7), g.get_links, lambda: g.set_launch(64, 0, 2), lambda: g.sweep_timed(5.7),
                 lambda: g.autotune(5), lambda: g.plaquette(5.7)):
        with pytest.raises(su3hb.SU3HBError) as ei:
            call()
        assert ei.value.code == su3hb.EHIP
    su3hb.su3hb_set_wait_limit(g.handle, 1 << 24)
    g.set_links(links)
    assert np.array_equal(g.get_links(), links)
    g.set_state(9, 2)
    assert np.array_equal(g.sweep_measure(5.7, n_sweeps=3), ref.sweep_measure(5.7, n_sweeps=3), equal_nan=True)
    assert np.array_equal(g.get_links(), ref.get_links()) and g.get_state() == ref.get_state() == (9, 5)


def test_every_replica_of_a_batch_has_to_be_set():
    reps = [((4, 4, 4, 4), 5.5 + 0.2 * r, r + 1, su3hb.HOT) for r in range(3)]
    b, ref = (su3hb.Batch(4, reps, precision=su3hb.FP32_18) for _ in range(2))
    su3hb.su3hb_set_wait_limit(b._h, 1)
    b.sweep(n_sweeps=40)
    with pytest.raises(su3hb.SU3HBError):
        b.sweep(n_sweeps=1, mode=1)
    for r in range(3):
        with pytest.raises(su3hb.SU3HBError):
            b.plaquette()
        b.set_links(r, ref.get_links(r))
    assert np.array_equal(b.plaquette(), ref.plaquette(), equal_nan=True)
