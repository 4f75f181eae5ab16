"""The launch shape of a lattice for which none is set gives the links of every
other shape, whether or not its order applies to the extents."""
import numpy as np
import pytest

import paper_0904_0642_amd as su3hb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ext,nlat,prec", [
    ([16, 16, 16, 32], 1, su3hb.FP64_18), ([16, 16, 16, 32], 1, su3hb.FP32_18), ([16, 14, 18, 22], 1, su3hb.FP64_12),
    ([16, 12, 10, 22], 2, su3hb.FP32_18), ([34, 32, 64], 1, su3hb.FP32_12), ([260, 254], 1, su3hb.FP64_18),
    ([10, 8, 8, 8, 14], 1, su3hb.FP32_18)])
def test_default_shape_gives_the_same_links(ext, nlat, prec):
    a, b = (su3hb.Lattice(ext, nlat=nlat, dlt_mask=1 if nlat == 2 else 0, precision=prec, seed=3) for _ in range(2))
    b.set_launch(64, 0, 2)
    sa, sb = (g.sweep_measure(5.8, 6.0, n_sweeps=2) for g in (a, b))
    assert nlat * np.prod(ext) // 2 > 32768  # one thread per link
    assert np.array_equal(a.get_links(), b.get_links())
    assert np.allclose(sa, sb, rtol=1e-12, atol=0, equal_nan=True)
