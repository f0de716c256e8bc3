"""The block stencil takes a thread per cell on levels of up to 1,024 blocks and
one per two cells above: the same bits, norms included."""
import numpy as np
import pytest

import ohm_inputs as gen

from gpu_util import announce, cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("bb", [(9, 9, 9), (8, 8, 16)])
def test_both_launches(dtype, bb):
    import torch
    import paper_1009_0798_amd as ohm
    announce(f"stencil threads {dtype} {bb}")
    rng = np.random.default_rng(53)
    tdt = torch.float64 if dtype == "f64" else torch.float32
    ijk = gen.full_level(bb)
    nb = len(ijk)
    assert nb <= 1024 < 2 * nb
    B, S = (cuda(rng.standard_normal((3, nb, 8, 8, 8)), tdt) for _ in range(2))
    E = cuda(np.exp(rng.uniform(-1, 1, (1, nb, 8, 8, 8))), tdt)
    got = []
    for n in (1, 2):
        H = ohm.Hierarchy([(bb, 0.1, [ijk])] * n)
        b, s, e = (torch.cat([x] * n, dim=1) for x in (B, S, E))
        out, R, Q = torch.empty_like(b), torch.empty_like(b), b.clone()
        ohm.ohm_apply(H, 0, b, e, [0.02] * n, out)
        nrm = ohm.ohm_residual(H, 0, b, s, e, [0.02] * n, R=R, norms=True)
        ohm.ohm_smooth(H, 0, Q, s, e, [0.02] * n, 1, torch.empty_like(b), ordering=1)   # colour by colour
        got.append([x[:, :nb] for x in (out, R, Q)] + [nrm[0]])
        assert torch.equal(R[:, -nb:], got[-1][1]) and np.array_equal(nrm[-1], nrm[0])
    for x, y in zip(got[0][:3], got[1][:3]):
        assert torch.equal(x, y)
    assert np.array_equal(got[0][3], got[1][3])
