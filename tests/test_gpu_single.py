"""Handles of one problem pass no work list and no problem table to the small
kernels; their steps equal, bit for bit, those of the same problem within a
batch, which lists both."""
import numpy as np
import pytest

import ohm_inputs as gen

from gpu_util import announce, cuda, dense_to_blocks

pytestmark = pytest.mark.gpu


# one block across (cell-wise dense kernels), a coarsest grid of 5 x 3 x 7
# cells (315 unknowns: more than the columns held in registers, and no
# multiple of the slices), a tile-wise dense level with rows of 12 cells
@pytest.mark.parametrize("bb", [(2, 1, 1), (5, 3, 7), (6, 4, 10)])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nuc", [1, 2])
def test_single_equals_batch(bb, precision, nuc):
    import torch
    import paper_1009_0798_amd as ohm
    announce(f"single == batch {bb} precision {precision} nu_coarse {nuc}")
    rng = np.random.default_rng(17)
    ijk = gen.full_level(bb)
    n = [8 * b for b in bb]
    dx, dt = 0.05, 0.05 ** 2 * 30.0
    B = [cuda(rng.standard_normal((3, len(ijk), 8, 8, 8))) for _ in range(2)]
    E = [cuda(np.exp(rng.uniform(-1, 1, (1, len(ijk), 8, 8, 8)))) for _ in range(2)]
    opts = ohm.default_opts(rtol=1e-9, precision=precision, max_iters=60, nu_pre=2, nu_post=3, nu_coarse=nuc)
    both = torch.cat(B, dim=1)
    st, stats = ohm.ohm_cn_step(ohm.Hierarchy([(bb, dx, [ijk])] * 2), [both], [torch.cat(E, dim=1)], [dt, dt], opts)
    assert st == 0
    for i in range(2):
        b = B[i].clone()
        st, one = ohm.ohm_cn_step(ohm.Hierarchy([(bb, dx, [ijk])]), [b], [E[i]], dt, opts)
        assert st == 0 and one[0]["iters"] == stats[i]["iters"]
        assert torch.equal(b, both[:, i * len(ijk):(i + 1) * len(ijk)])
