"""The way down from dense levels of few tiles: the sweep from a zero guess, the
residual and its restriction in one launch (one sweep before the residual) or
the last two (more sweeps), on parts of the tiles.  A large enough batch of the
same problem takes the separate kernels of whole tiles; steps of both are equal
bit for bit, and so are those of a V-cycle without these launches on the
base level."""
import numpy as np
import pytest

import ohm_inputs as gen

from gpu_util import announce, cuda

pytestmark = pytest.mark.gpu


# dense levels of 30 tiles that overhang the grid (quarters alone, halves and
# whole tiles in the batches); of 27; of 4 tiles with edges of 4 cells and, one
# level below, of 2 (the separate kernels)
@pytest.mark.parametrize("bb,counts", [((6, 4, 10), (1, 3, 5)), ((5, 5, 5), (1, 3, 5)), ((8, 1, 1), (1, 20, 70))])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nuc", [1, 2])
def test_way_down(bb, counts, precision, nuc):
    import torch
    import paper_1009_0798_amd as ohm
    announce(f"way down {bb} precision {precision} nu_coarse {nuc}")
    rng = np.random.default_rng(43)
    ijk = gen.full_level(bb)
    dx, dt = 0.05, 0.05 ** 2 * 30.0
    b0 = cuda(rng.standard_normal((3, len(ijk), 8, 8, 8)))
    e0 = cuda(np.exp(rng.uniform(-1, 1, (1, len(ijk), 8, 8, 8))))
    opts = ohm.default_opts(rtol=1e-9, precision=precision, max_iters=60, nu_pre=2, nu_post=3, nu_coarse=nuc)
    got = []
    for n in counts:
        b = torch.cat([b0] * n, dim=1)
        H = ohm.Hierarchy([(bb, dx, [ijk])] * n)
        st, stats = ohm.ohm_cn_step(H, [b], [torch.cat([e0] * n, dim=1)], [dt] * n, opts)
        assert st == 0
        got.append((b[:, :len(ijk)], stats[0]["iters"]))
        assert torch.equal(b[:, -len(ijk):], got[-1][0])
    for b, it in got[1:]:
        assert it == got[0][1] and torch.equal(b, got[0][0])
