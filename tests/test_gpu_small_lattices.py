"""Small lattices and batches, whose slices share every link's update between
lanes and waves, and (up to 64 groups of 16 links) whose calls run whole
sweeps in one launch: the same bits as one thread per link (a launch shape set
by the caller), at the edges of the groups and of the two forms' ranges."""
import numpy as np
import pytest

import paper_0904_0642_amd as su3hb

pytestmark = pytest.mark.gpu

P = (su3hb.FP64_18, su3hb.FP32_18, su3hb.FP32_12, su3hb.FP64_12)


def pair(ext, prec, nlat=1, mask=0, **kw):
    a, b = (su3hb.Lattice(ext, nlat=nlat, dlt_mask=mask, precision=prec, seed=17, **kw) for _ in range(2))
    b.set_launch(256, 1, 2)
    return a, b


def same_counters(x, y, scale):
    assert {k: v for k, v in x.items() if k != "dtrace"} == {k: v for k, v in y.items() if k != "dtrace"}
    # a sum over the links in another order: rounding of terms of order `scale`
    assert abs(x["dtrace"] - y["dtrace"]) <= 1e-12 * scale


@pytest.mark.parametrize("prec", P)
@pytest.mark.parametrize("ext,nlat,mask", [
    ([2, 2], 1, 0), ([4, 8], 1, 0), ([6, 6], 2, 0b11), ([32, 64], 1, 0),      # 2, 16, 2 x 18, 1024 links
    ([2, 2, 4], 1, 0), ([6, 4, 10], 2, 0b101), ([30, 22, 18], 1, 0),          # 8, 2 x 120, 5940 links
    ([4, 4, 4, 4], 1, 0), ([8, 8, 8, 4], 1, 0), ([2, 2, 2, 258], 1, 0),       # 128, 1024, 1032 links
    ([6, 4, 4, 4], 2, 0b0111), ([10, 6, 4, 10], 2, 0b1111),                   # 2 x 192, 2 x 1200 links
    ([4, 2, 6, 2, 4], 1, 0), ([4, 4, 4, 6, 6], 2, 0b11111),                   # 192, 2 x 1152 links
    ([2, 4, 2, 2, 4, 2], 1, 0), ([4, 4, 2, 4, 4, 6], 1, 0),                   # 128, 1536 links
])
def test_shared_updates_give_the_same_links(ext, nlat, mask, prec):
    a, b = pair(ext, prec, nlat, mask)
    nplaq = a.n_links * (len(ext) - 1) / 2
    for n in (1, 2):
        (sa, ta), (sb, tb) = (g.sweep_measure(5.5, 6.1, n_hit=8, n_sweeps=n, stats=True) for g in (a, b))
        assert np.array_equal(a.get_links(), b.get_links())
        same_counters(ta, tb, 6.1 * nplaq)
        # averages of at most nplaq numbers below 1, and their beta-weighted sum
        assert np.allclose(sa[:, :5], sb[:, :5], rtol=1e-12, atol=1e-13, equal_nan=True)
        assert np.allclose(sa[:, 5], sb[:, 5], rtol=1e-12, atol=1e-13 * 6.1 * nplaq)
        a.overrelax(5.5, 6.1, n_sweeps=1)
        b.overrelax(5.5, 6.1, n_sweeps=1)
    assert np.array_equal(a.get_links(), b.get_links()) and a.get_state() == b.get_state()


@pytest.mark.parametrize("ext", [[4, 4, 4, 4], [12, 8, 8, 6]])
@pytest.mark.parametrize("beta,n_hit", [(5.7, 1), (5.7, 2), (-2.0, 8), (0.3, 200), (1.5, 6), (0.0, 3)])
def test_rejected_proposals(ext, beta, n_hit):
    # first hits, second hits (both drawn ahead), later ones (four at a time),
    # all rejected, and a degenerate projection
    for prec in (su3hb.FP64_18, su3hb.FP32_12):
        a, b = pair(ext, prec)
        ta, tb = (g.sweep(beta, n_hit=n_hit, n_sweeps=2, stats=True) for g in (a, b))
        assert np.array_equal(a.get_links(), b.get_links())
        same_counters(ta, tb, 6.0 * a.n_links * max(1.0, abs(beta)))


def test_identical_random_numbers_on_two_layers():
    a, b = (su3hb.Lattice([4, 4, 4, 6], nlat=2, lat2test=True, seed=9) for _ in range(2))
    b.set_launch(128, 0, 2)
    for g in (a, b):
        g.sweep(5.8, n_sweeps=3)
    links = a.get_links()
    assert np.array_equal(links, b.get_links()) and np.array_equal(links[0], links[1])


@pytest.mark.parametrize("prec", (su3hb.FP64_18, su3hb.FP32_18))
@pytest.mark.parametrize("shapes", [[(4, 4, 4, 4)] * 3, [(2, 4, 2, 6), (4, 4, 4, 4), (6, 4, 2, 2), (2, 2, 2, 2)],
                                    [(8, 8, 6, 4), (6, 10, 4, 4), (4, 4, 4, 4)]])
def test_batches(shapes, prec):
    reps = [(s, 5.5 + 0.1 * i, 40 + i, su3hb.HOT) for i, s in enumerate(shapes)]
    a, b, c = (su3hb.Batch(4, reps, precision=prec) for _ in range(3))
    b.set_launch(64, 0, 2)
    ta, tb = (g.sweep(n_hit=8, n_sweeps=3, stats=True) for g in (a, b))
    c.sweep(n_hit=8, n_sweeps=3, mode=1)
    same_counters(ta, tb, 6.0 * a.links_per_sweep * 3 * 6.5)
    for r in range(len(reps)):
        assert np.array_equal(a.get_links(r), b.get_links(r)) and np.array_equal(a.get_links(r), c.get_links(r))


def test_forms_alternate_on_one_lattice():
    # whole sweeps in one launch, then slice by slice in a set shape, then with
    # the tuner's choice: one chain, one sweep counter
    a = su3hb.Lattice([6, 4, 4, 4], seed=2)
    b = su3hb.Lattice([6, 4, 4, 4], seed=2)
    b.set_launch(64, 0, 2)
    for k in range(3):
        a.sweep(5.9, n_sweeps=2)
        _, sa = a.sweep_timed(5.9, n_sweeps=2, measure=True)
        a.set_launch(128, 1, 2)
        a.sweep(5.9, n_sweeps=1)
        a.autotune(20)
        sa2 = a.sweep_measure(5.9, n_sweeps=2)
        b.sweep(5.9, n_sweeps=2)
        _, sb = b.sweep_timed(5.9, n_sweeps=2, measure=True)
        b.sweep(5.9, n_sweeps=1)
        sb2 = b.sweep_measure(5.9, n_sweeps=2)
        assert np.array_equal(a.get_links(), b.get_links()), k
        assert np.allclose(sa, sb, rtol=1e-12, atol=0, equal_nan=True)
        assert np.allclose(sa2, sb2, rtol=1e-12, atol=0, equal_nan=True)
    assert a.get_state() == b.get_state() == (2, 21)


def test_many_launches_take_queue_after_queue():
    # more launches of whole sweeps than there are queues between two clearings
    a, b = (su3hb.Lattice([4, 4, 2, 4], seed=5) for _ in range(2))
    parts = [a.sweep_measure(5.7, n_sweeps=1) if k % 3 else a.sweep(5.7, n_sweeps=1) for k in range(150)]
    b.sweep_measure(5.7, n_sweeps=150)
    assert np.array_equal(a.get_links(), b.get_links()) and a.get_state() == b.get_state()
    assert np.array_equal(a.sweep_measure(5.7, n_sweeps=2), b.sweep_measure(5.7, n_sweeps=2), equal_nan=True)
    assert all(p is None or p.shape == (1, 6) for p in parts)


def test_lattices_on_two_streams():
    # two lattices whose launches may run side by side keep their queues apart
    import torch
    ref, out = [], []
    for seed in (3, 4):
        g = su3hb.Lattice([8, 4, 4, 4], seed=seed)
        g.sweep(5.8, n_sweeps=40)
        ref.append(g.get_links())
    streams = [torch.cuda.Stream() for _ in range(2)]
    lats = []
    for s, seed in zip(streams, (3, 4)):
        with torch.cuda.stream(s):
            lats.append(su3hb.Lattice([8, 4, 4, 4], seed=seed))
    for _ in range(4):
        for g in lats:
            g.sweep(5.8, n_sweeps=10)
    out = [g.get_links() for g in lats]
    assert all(np.array_equal(x, y) for x, y in zip(ref, out))
