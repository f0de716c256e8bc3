"""The marching operator of large base levels: against the oracle on boxes whose
edges are not multiples of the 16-cell tiles, and bit for bit against the
operator per 8^3 block, which a residual with norms takes.  (Its fused dot
products and restriction are compared with those of the operator per block by
the steps of the marching batch.)"""
import numpy as np
import pytest

import ohm_inputs as gen
from oracle import ref

from gpu_util import announce, blocks_to_dense, cuda, dense_to_blocks, hier, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bb", [(17, 13, 21), (2, 33, 64), (16, 16, 16)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_marching_operator(bb, dtype):
    import torch
    import paper_1009_0798_amd as ohm
    announce(f"marching operator {bb} {dtype}")
    spec = gen.HierSpec(bb, 0.05, [gen.full_level(bb)])
    nx, ny, nz = spec.cells(0)
    rng = np.random.default_rng(41)
    tdt = torch.float64 if dtype == "f64" else torch.float32
    B, S = rng.standard_normal((3, nz, ny, nx)), rng.standard_normal((3, nz, ny, nx))
    eta = np.exp(np.log(10.0) * rng.uniform(-1, 1, (nz, ny, nx)))
    if dtype == "f32":
        B, S, eta = (x.astype(np.float32).astype(np.float64) for x in (B, S, eta))
    ijk = spec.levels[0]
    H = hier(spec)
    lam_dt = 10.0 * spec.dx0 ** 2 / eta.max()
    Bt, St, Et = (cuda(dense_to_blocks(a, ijk), tdt) for a in (B, S, eta[None]))
    # about 40 rounded terms a cell, as for the operator per block
    scale = np.abs(B).max() * (1.0 + 16.0 * lam_dt * eta.max() / spec.dx0 ** 2)
    tol = (5e-14 if dtype == "f64" else 2e-5) * scale
    out = torch.full_like(Bt, float("nan"))
    ohm.ohm_apply(H, 0, Bt, Et, lam_dt, out)
    assert np.abs(blocks_to_dense(host(out), ijk, spec.cells(0)) - ref.apply(B, eta, spec.dx0, lam_dt)).max() <= tol
    blk, R = torch.full_like(Bt, float("nan")), torch.full_like(Bt, float("nan"))
    ohm.ohm_residual(H, 0, Bt, St, Et, lam_dt, R=blk, norms=True)
    ohm.ohm_residual(H, 0, Bt, St, Et, lam_dt, R=R)
    assert np.abs(blocks_to_dense(host(R), ijk, spec.cells(0)) - ref.residual(B, S, eta, spec.dx0, lam_dt)).max() <= tol
    assert torch.equal(R, blk)
    ohm.ohm_residual(H, 0, Bt, St, Et, lam_dt, R=St)   # in place of S
    assert torch.equal(St, blk)
