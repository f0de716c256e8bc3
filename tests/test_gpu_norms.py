"""The norms of a residual: sums and maxima of the residual it writes, over
blocks of both launches of the stencil, also where values are not finite."""
import numpy as np
import pytest

import ohm_inputs as gen

from gpu_util import announce, cuda, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("bb", [(1, 1, 1), (3, 5, 2), (10, 10, 11)])
def test_norms_of_the_written_residual(dtype, bb):
    import torch
    import paper_1009_0798_amd as ohm
    announce(f"norms {dtype} {bb}")
    rng = np.random.default_rng(71)
    tdt = torch.float64 if dtype == "f64" else torch.float32
    ijk = gen.full_level(bb)
    nb = len(ijk)
    H = ohm.Hierarchy([(bb, 0.1, [ijk])])
    B, S = (cuda(rng.standard_normal((3, nb, 8, 8, 8)) * 10.0 ** rng.uniform(-3, 3, (3, nb, 1, 1, 1)), tdt) for _ in range(2))
    E = cuda(np.exp(rng.uniform(-1, 1, (1, nb, 8, 8, 8))), tdt)
    R = torch.empty_like(B)

    def norms():
        n = ohm.ohm_residual(H, 0, B, S, E, 0.02, R=R, norms=True)[0]
        return n, host(R).reshape(3, -1)

    n, r = norms()
    # sums of 512 nb squares: at most that many roundings of 2^-53
    assert (np.abs(n[:, 0] / np.array([np.sum(c.astype(np.longdouble) ** 2) for c in r]) - 1) <= 512 * nb * 2.0 ** -53).all()
    assert (n[:, 1] == np.abs(r).max(axis=1)).all()
    # a value that is no number makes the sum none and leaves the maximum alone
    S[1, nb // 2, 7, 3, 5] = float("nan")
    S[2, nb - 1, 0, 0, 7] = float("-inf")
    n, r = norms()
    assert np.isfinite(n[0]).all() and np.isnan(n[1, 0]) and n[1, 1] == np.nanmax(np.abs(r[1])) and (n[2] == np.inf).all()
