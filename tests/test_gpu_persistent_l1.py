"""Persistent batch sweeps whose last blocks hold few links: all such a block
reads in a slice stays in its compute unit's L1, so every slice must begin with
an L1 that holds nothing of the slices before.  Against one launch per slice."""
import numpy as np
import pytest
import torch  # noqa: F401 -- its HIP runtime is the one to load

import paper_0904_0642_amd as su3hb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", (su3hb.FP64_18, su3hb.FP32_18, su3hb.FP32_12, su3hb.FP64_12))
@pytest.mark.parametrize("shape", [(2, 2, 2, 66), (6, 4, 2, 12), (258, 4), (8, 66), (4, 4, 4, 18)])
def test_short_last_blocks(shape, prec):
    reps = [(shape, 5.7, r + 1, su3hb.HOT) for r in range(16)]
    a, b = (su3hb.Batch(len(shape), reps, precision=prec) for _ in range(2))
    a.sweep(n_hit=8, n_sweeps=20, mode=1)
    b.sweep(n_hit=8, n_sweeps=20, mode=0)
    assert all(np.array_equal(a.get_links(r), b.get_links(r)) for r in range(len(reps)))
