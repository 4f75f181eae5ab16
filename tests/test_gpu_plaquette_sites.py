"""The plaquette launch for 65536 sites and more (one thread per site) against
the oracle's plaquettes of the same links: whole and ragged tiles of the
half-lattice, every dimension, two layers, batches of several shapes; and just
below the line, where each thread has a (site, plane)."""
import numpy as np
import pytest

import paper_0904_0642_amd as su3hb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ext,nlat,mask,prec", [
    ([256, 256], 1, 0, su3hb.FP64_18), ([14, 4682], 1, 0, su3hb.FP32_18),          # 65536, 65548 sites
    ([42, 38, 42], 1, 0, su3hb.FP64_12), ([34, 30, 34], 2, 0b101, su3hb.FP32_12),  # 67032, 2 x 34680
    ([16, 16, 16, 16], 1, 0, su3hb.FP32_12), ([18, 14, 14, 20], 1, 0, su3hb.FP64_18),
    ([14, 12, 14, 14], 2, 0b1111, su3hb.FP64_12), ([16, 16, 16, 14], 1, 0, su3hb.FP64_18),  # 57344: below
    ([10, 10, 10, 10, 8], 1, 0, su3hb.FP32_18), ([6, 6, 6, 6, 8, 8], 1, 0, su3hb.FP64_18),
])
def test_plaquette_matches_oracle(oracle_mod, ext, nlat, mask, prec):
    g = su3hb.Lattice(ext, nlat=nlat, dlt_mask=mask, precision=prec, seed=6)
    g.sweep(5.0, 5.6, n_hit=2)
    o = oracle_mod.Lattice(ext, nlat=nlat, dlt_mask=mask, seed=6)
    o.set_links(g.get_links())
    got, want = g.plaquette(5.0, 5.6), o.plaquette(5.0, 5.6)
    # averages of numbers below 1 over the same links, formed in FP64 on both
    # sides (12-real FP32 links: the third row is the one get_links returned)
    n = nlat * np.prod(ext) * len(ext) * (len(ext) - 1) / 2
    assert np.allclose(got[:5], want[:5], rtol=1e-12, atol=1e-13, equal_nan=True)
    assert abs(got[5] - want[5]) <= 1e-13 * 5.6 * n
    assert np.array_equal(g.plaquette(5.0, 5.6), got, equal_nan=True)


def test_batch_of_several_shapes(oracle_mod):
    shapes = [(16, 12, 12, 12), (6, 4, 2, 10), (14, 14, 14, 14), (2, 2, 2, 2)]  # 65 960 sites
    reps = [(s, 5.5 + 0.2 * i, 5 + i, su3hb.HOT) for i, s in enumerate(shapes)]
    b = su3hb.Batch(4, reps, precision=su3hb.FP32_18)
    got = b.plaquette()
    for r, (s, beta, seed, _) in enumerate(reps):
        o = oracle_mod.Lattice(list(s), seed=seed)
        o.set_links(b.get_links(r))
        assert np.allclose(got[r], o.plaquette(beta), rtol=1e-12, atol=1e-13, equal_nan=True), s


@pytest.mark.parametrize("ext,nlat,mask,prec", [
    ([16, 12, 12, 30], 1, 0, su3hb.FP64_18), ([32, 2, 4, 258], 1, 0, su3hb.FP32_18),      # three strips; one of one tile
    ([16, 8, 20, 26], 2, 0b1010, su3hb.FP32_12), ([16, 16, 18, 16], 1, 0, su3hb.FP64_12),  # two layers; a cut strip
    ([14, 10, 20, 24], 1, 0, su3hb.FP32_18),                                              # rows that cut a tile
    ([8, 8, 4, 8, 32], 1, 0, su3hb.FP64_12), ([4, 4, 4, 4, 8, 32], 1, 0, su3hb.FP32_12),
])
def test_strips_take_every_site_once(oracle_mod, ext, nlat, mask, prec):
    g = su3hb.Lattice(ext, nlat=nlat, dlt_mask=mask, precision=prec, seed=9)
    o = oracle_mod.Lattice(ext, nlat=nlat, dlt_mask=mask, seed=9)
    o.set_links(g.get_links())
    # a site taken twice for another changes the averages by 1 / (number of
    # plaquettes), above 1e-7 here; rounding stays below 1e-12
    assert np.allclose(g.plaquette(5.0, 5.6)[:5], o.plaquette(5.0, 5.6)[:5], rtol=1e-12, atol=1e-13, equal_nan=True)
