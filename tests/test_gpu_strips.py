"""Runs of blocks in strips of x_{D-2} along x_{D-1} (lattices whose x_{D-1}
steps pass an XCD's L2): the same bits as blocks in hardware order, with rows
and runs that end anywhere, two layers, every block size and the staging of
neighbours; and lattices just outside the rule."""
import numpy as np
import pytest

import paper_0904_0642_amd as su3hb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ext,nlat,mask,prec", [
    ([24, 24, 20, 10], 1, 0, su3hb.FP64_18), ([24, 24, 24, 8], 2, 0b1111, su3hb.FP32_18),  # 6.3 MB, 2 x 3.8 MB a step
    ([16, 20, 24, 10], 2, 0b0110, su3hb.FP64_12), ([36, 32, 28, 6], 1, 0, su3hb.FP32_12),  # 2 x 2.8 MB, 5.9 MB
    ([16, 10, 32, 14], 2, 0b1001, su3hb.FP64_18), ([16, 10, 68, 10], 1, 0, su3hb.FP64_18),  # the last: 850 waves, a cut block
    ([320, 320, 6], 1, 0, su3hb.FP64_18), ([32, 1796, 4], 1, 0, su3hb.FP32_18),  # rows of ten waves and of one
    ([24, 24, 22, 10], 1, 0, su3hb.FP64_18), ([22, 22, 24, 10], 1, 0, su3hb.FP64_18),  # no whole strips; cut waves
])
def test_strips_take_every_link_once(ext, nlat, mask, prec):
    a, b = (su3hb.Lattice(ext, nlat=nlat, dlt_mask=mask, precision=prec, seed=8) for _ in range(2))
    b.set_launch(64, 0, 2)
    # staging areas of 320-site rows pass the LDS and are refused
    shapes = [(256, 1), (128, 9), (64, 1)] + ([(256, 17), (64, 25)] if nlat == 1 and ext[0] < 64 else [])
    for block, order in shapes:
        a.set_launch(block, order, 2)
        assert a.get_launch()[1] == order
        sa, sb = (g.sweep_measure(5.5, 6.1, n_hit=8, n_sweeps=1) for g in (a, b))
        assert np.array_equal(a.get_links(), b.get_links()), (block, order)
        assert np.allclose(sa, sb, rtol=1e-12, atol=1e-13, equal_nan=True)
