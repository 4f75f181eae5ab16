"""Middle-sized lattices and batches, whose slices give the planes of a link's
staple to waves of their own: the same bits as one thread per link (a launch
shape set by the caller), at the edges of that form's range, with ragged last
blocks, on two layers and in batches."""
import numpy as np
import pytest

import paper_0904_0642_amd as su3hb

pytestmark = pytest.mark.gpu

F64, F32, F32_12, F64_12 = su3hb.FP64_18, su3hb.FP32_18, su3hb.FP32_12, su3hb.FP64_12


def pair(ext, prec, nlat=1, mask=0, **kw):
    a, b = (su3hb.Lattice(ext, nlat=nlat, dlt_mask=mask, precision=prec, seed=17, **kw) for _ in range(2))
    b.set_launch(256, 1, 2)
    return a, b


def same_counters(x, y, scale):
    assert {k: v for k, v in x.items() if k != "dtrace"} == {k: v for k, v in y.items() if k != "dtrace"}
    # a sum over the links in another order: rounding of terms of order `scale`
    assert abs(x["dtrace"] - y["dtrace"]) <= 1e-12 * scale


@pytest.mark.parametrize("ext,nlat,mask,prec", [
    ([16, 16, 16, 10], 1, 0, F64), ([2, 2, 6, 1708], 1, 0, F64),              # 20480, 20496 links: the lower line
    ([14, 14, 14, 18], 1, 0, F64_12), ([14, 14, 14, 18], 1, 0, F32),          # 24696: a cut last block
    ([16, 16, 16, 16], 1, 0, F64), ([16, 16, 16, 18], 1, 0, F64),             # 512 blocks and above
    ([24, 16, 16, 16], 1, 0, F32_12), ([16, 12, 16, 34], 1, 0, F32),          # 768 blocks and above
    ([10, 14, 12, 14], 2, 0b1111, F64), ([12, 12, 12, 14], 2, 0b0101, F32_12),  # 2 x 11760, 2 x 12096
    ([14, 10, 14, 12], 2, 0b1000, F64_12), ([12, 14, 14, 16], 2, 0b0011, F32),  # 2 x 11760, 2 x 18816
    ([34, 38, 38], 1, 0, F64), ([42, 34, 36], 1, 0, F32_12),                  # 24548, 25704
    ([34, 30, 28], 2, 0b101, F64), ([48, 32, 64], 1, 0, F32),                 # 2 x 14280, 49152
    ([16, 12, 16, 18], 2, 0b0110, F32), ([48, 34, 64], 1, 0, F32_12),         # 2 x 27648, 52224: a thread per link
])
def test_planes_on_waves_give_the_same_links(ext, nlat, mask, prec):
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


@pytest.mark.parametrize("ext", [[14, 14, 14, 16], [32, 32, 50]])
@pytest.mark.parametrize("beta,n_hit", [(5.7, 1), (5.7, 2), (-2.0, 8), (0.3, 200), (1.5, 6), (0.0, 3)])
def test_rejected_proposals(ext, beta, n_hit):
    # first hits, second hits (both drawn ahead), later ones, all rejected, and
    # a degenerate projection
    for prec in (F64, F32_12):
        a, b = pair(ext, prec)
        ta, tb = (g.sweep(beta, n_hit=n_hit, n_sweeps=2, stats=True) for g in (a, b))
        assert np.array_equal(a.get_links(), b.get_links())
        same_counters(ta, tb, 6.0 * a.n_links * max(1.0, abs(beta)))


@pytest.mark.parametrize("prec", (F64, F32))
def test_batches(prec):
    shapes = [(14, 14, 14, 14), (6, 4, 2, 10), (12, 12, 12, 4), (2, 2, 2, 2)]  # 22912 links in a slice
    reps = [(s, 5.5 + 0.1 * i, 40 + i, su3hb.HOT) for i, s in enumerate(shapes)]
    a, b = (su3hb.Batch(4, reps, precision=prec) for _ in range(2))
    b.set_launch(64, 0, 2)
    ta, tb = (g.sweep(n_hit=8, n_sweeps=3, stats=True) for g in (a, b))
    same_counters(ta, tb, 6.0 * a.links_per_sweep * 3 * 6.5)
    for r in range(len(reps)):
        assert np.array_equal(a.get_links(r), b.get_links(r))


def test_random_numbers_of_two_layers_and_forms_alternate():
    a, b = (su3hb.Lattice([10, 12, 14, 14], nlat=2, lat2test=True, seed=9) for _ in range(2))
    b.set_launch(128, 0, 2)
    for g in (a, b):
        g.sweep(5.8, n_sweeps=2)
    links = a.get_links()
    assert np.array_equal(links, b.get_links()) and np.array_equal(links[0], links[1])
    a, b = (su3hb.Lattice([14, 14, 14, 16], seed=2) for _ in range(2))
    b.set_launch(64, 0, 2)
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
    assert np.array_equal(a.get_links(), b.get_links())
    assert np.allclose(sa, sb, rtol=1e-12, atol=0, equal_nan=True)
    assert np.allclose(sa2, sb2, rtol=1e-12, atol=0, equal_nan=True)
    assert a.get_state() == b.get_state() == (2, 7)


@pytest.mark.parametrize("ext", [[4, 4, 4, 4], [14, 14, 14, 16], [24, 24, 20, 10]])
def test_static_sweeps_in_a_captured_graph(ext):
    # every form of a slice, replayed with work between the replays, against
    # the same calls one by one
    import ctypes as C

    import torch

    def call(lat, series, stream):
        p = su3hb.make_params(ext, 1, 0, False, F64, su3hb.HOT, 5, device_links=C.c_void_p(lat.buffer.data_ptr()),
                              device_bytes=lat.buffer.numel(), hip_stream=C.c_void_p(stream.cuda_stream))
        su3hb.su3hb_sweep_measure_static(p, 5.9, 5.9, 8, 2, 0, C.c_void_p(series.data_ptr()))

    a, b = (su3hb.Lattice(ext, seed=5) for _ in range(2))
    sa, sb = (torch.zeros(12, dtype=torch.float64, device="cuda") for _ in range(2))
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    call(a, sa, s)  # looks the scratch up
    call(b, sb, s)
    s.synchronize()
    with torch.cuda.stream(s):
        graph = torch.cuda.CUDAGraph()
        graph.capture_begin()
        call(a, sa, s)
        graph.capture_end()
        for _ in range(4):
            graph.replay()
            s.synchronize()
            torch.ones(1000, device="cuda").sum().item()
            call(b, sb, s)
            s.synchronize()
            assert torch.equal(sa.nan_to_num(-1.0), sb.nan_to_num(-1.0))
            assert torch.equal(a.buffer, b.buffer)
