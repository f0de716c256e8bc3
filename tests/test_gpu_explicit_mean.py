"""The explicit step of a one-level handle averages in the second application:
equal, bit for bit, to the two applications and the mean taken one by one."""
import numpy as np
import pytest

import ohm_inputs as gen

from gpu_util import announce, cuda

pytestmark = pytest.mark.gpu


# one block; a ragged box; a base level of a few thousand blocks
@pytest.mark.parametrize("bb", [(1, 1, 1), (5, 3, 7), (17, 13, 21)])
@pytest.mark.parametrize("nsteps", [1, 3])
def test_explicit_step_equals_its_parts(bb, nsteps):
    import torch
    import paper_1009_0798_amd as ohm
    announce(f"explicit mean {bb} {nsteps}")
    rng = np.random.default_rng(37)
    ijk = gen.full_level(bb)
    dx, dt = 0.1, 0.1 ** 2 * 0.03
    x = cuda(rng.standard_normal((3, len(ijk), 8, 8, 8)))
    e = cuda(np.exp(rng.uniform(-1, 1, (1, len(ijk), 8, 8, 8))))
    H = ohm.Hierarchy([(bb, dx, [ijk])])
    got = x.clone()
    ohm.ohm_explicit_step(H, [got], [e], dt, nsteps)
    p, v = torch.empty_like(x), torch.empty_like(x)
    for _ in range(nsteps):
        ohm.ohm_apply(H, 0, x, e, -dt, p)
        ohm.ohm_apply(H, 0, p, e, -dt, v)
        x = 0.5 * (x + v)
    assert torch.isfinite(x).all() and torch.equal(got, x)
