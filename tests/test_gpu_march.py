"""The marching sweeps of large base levels (boxes and handles of a few thousand
blocks): against the oracle on boxes whose edges are not multiples of the
16-cell tiles, and bit for bit against the sweep per 8^3 block that the same
problems take when they are solved alone."""
import numpy as np
import pytest

import ohm_inputs as gen
from oracle import ref

from gpu_util import announce, blocks_to_dense, cuda, dense_to_blocks, hier, host

pytestmark = pytest.mark.gpu


def _eta(rng, shape):
    return np.exp(np.log(10.0) * rng.uniform(-1, 1, shape))


# 17 x 13 x 21 blocks: tiles of one block at both upper edges, a short last
# segment; 2 x 33 x 64: one tile across; 16^3: whole tiles
@pytest.mark.parametrize("bb", [(17, 13, 21), (2, 33, 64), (16, 16, 16)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_marching_sweep_against_oracle(bb, dtype):
    import torch
    import paper_1009_0798_amd as ohm
    announce(f"marching sweep {bb} {dtype}")
    spec = gen.HierSpec(bb, 0.05, [gen.full_level(bb)])
    nx, ny, nz = spec.cells(0)
    rng = np.random.default_rng(31)
    tdt = torch.float64 if dtype == "f64" else torch.float32
    B, S = rng.standard_normal((3, nz, ny, nx)), rng.standard_normal((3, nz, ny, nx))
    eta = _eta(rng, (nz, ny, nx))
    if dtype == "f32":
        B, S, eta = (x.astype(np.float32).astype(np.float64) for x in (B, S, eta))
    ijk = spec.levels[0]
    H = hier(spec)
    lam_dt = 10.0 * spec.dx0 ** 2 / eta.max()
    Bt, St, Et = (cuda(dense_to_blocks(a, ijk), tdt) for a in (B, S, eta[None]))
    ohm.ohm_smooth(H, 0, Bt, St, Et, lam_dt, 2, torch.empty_like(Bt))
    got = blocks_to_dense(host(Bt), ijk, spec.cells(0))
    ex = ref.smooth(B, S, eta, spec.dx0, lam_dt, 2)
    # as for the sweep per block: about 40 rounded terms per half-sweep
    scale = np.abs(B).max() * (1.0 + 16.0 * lam_dt * eta.max() / spec.dx0 ** 2)
    assert np.abs(got - ex).max() <= 8 * (5e-14 if dtype == "f64" else 2e-5) * scale


@pytest.mark.parametrize("precision", [0, 1])
def test_marching_batch_equals_alone(precision):
    """Zero-guess, plain and FP64-output sweeps inside a step: a handle large
    enough to march against the same problems alone (sweep per block)."""
    import torch
    import paper_1009_0798_amd as ohm
    announce(f"marching batch == alone, precision {precision}")
    specs = [gen.uniform_spec(n) for n in [40, 24, 32, 48, 16] * 11]
    assert sum(len(s.levels[0]) for s in specs) > 4000
    rng = np.random.default_rng(5)
    B = [torch.from_numpy(dense_to_blocks(gen.divfree(s.cells(0)[0], 2.0, seed=i), s.levels[0])) for i, s in enumerate(specs)]
    E = [torch.from_numpy(dense_to_blocks(gen.lognormal_eta(s.cells(0)[0], 2.0, seed=99 + i)[None], s.levels[0]))
         for i, s in enumerate(specs)]
    dts = [gen.explicit_dt(s.dx0, 1.0, float(rng.uniform(20, 80))) for s in specs]
    opts = ohm.default_opts(rtol=1e-10, precision=precision, max_iters=100, nu_pre=2, nu_post=3, nu_coarse=1)
    H = ohm.Hierarchy([(s.base_blocks, s.dx0, s.levels) for s in specs])
    Bt = torch.cat(B, dim=1).cuda()
    st, stats = ohm.ohm_cn_step(H, [Bt], [torch.cat(E, dim=1).cuda()], dts, opts)
    assert st == 0
    got = Bt.cpu()
    off = 0
    for i, s in enumerate(specs):
        nb = len(s.levels[0])
        if i < 10:
            b = B[i].cuda()
            st, one = ohm.ohm_cn_step(ohm.Hierarchy([(s.base_blocks, s.dx0, s.levels)]), [b], [E[i].cuda()], dts[i], opts)
            assert st == 0 and one[0]["iters"] == stats[i]["iters"]
            assert torch.equal(b.cpu(), got[:, off:off + nb]), i
        off += nb
