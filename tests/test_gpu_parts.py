"""Launches over few 8^3 tiles split each tile over two or four groups; a batch
of the same problem has more tiles and splits them less.  Steps of both are
equal bit for bit: sweeps (plain, from zero, with the coarse correction, to
FP64, next to coarse-fine ghost blocks) on base, refined and dense levels."""
import numpy as np
import pytest

import ohm_inputs as gen

from gpu_util import announce, cuda, dense_to_blocks

pytestmark = pytest.mark.gpu


# 64, 125 and 128 tiles alone (4, 2 and 2 parts), twice and five times as many
# in the batch (2, 1 and 1 parts; whole)
@pytest.mark.parametrize("bb", [(4, 4, 4), (5, 5, 5), (4, 4, 8)])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nu", [(2, 3), (3, 2)])
def test_parts_equal_whole_tiles(bb, precision, nu):
    import torch
    import paper_1009_0798_amd as ohm
    announce(f"parts {bb} precision {precision} nu {nu}")
    rng = np.random.default_rng(23)
    ijk = gen.full_level(bb)
    dx, dt = 0.05, 0.05 ** 2 * 30.0
    b0 = cuda(rng.standard_normal((3, len(ijk), 8, 8, 8)))
    e0 = cuda(np.exp(rng.uniform(-1, 1, (1, len(ijk), 8, 8, 8))))
    opts = ohm.default_opts(rtol=1e-9, precision=precision, max_iters=60, nu_pre=nu[0], nu_post=nu[1])
    got = []
    for n in (1, 2, 5):
        b = torch.cat([b0] * n, dim=1)
        H = ohm.Hierarchy([(bb, dx, [ijk])] * n)
        st, stats = ohm.ohm_cn_step(H, [b], [torch.cat([e0] * n, dim=1)], [dt] * n, opts)
        assert st == 0
        got.append((b[:, :len(ijk)], stats[0]["iters"]))
        assert torch.equal(b[:, -len(ijk):], got[-1][0])
    for b, it in got[1:]:
        assert it == got[0][1] and torch.equal(b, got[0][0])


@pytest.mark.parametrize("precision", [0, 1])
def test_parts_equal_whole_tiles_with_ghosts(precision):
    import torch
    import paper_1009_0798_amd as ohm
    announce(f"parts with ghosts, precision {precision}")
    spec = gen.config_amr2(n_base=32, extra_frac=0.0)
    assert 8 * len(spec.levels[1]) > 256
    rng = np.random.default_rng(29)
    lv = spec.levels
    B = [cuda(rng.standard_normal((3, len(l), 8, 8, 8))) for l in lv]
    E = [cuda(np.exp(rng.uniform(-1, 1, (1, len(l), 8, 8, 8)))) for l in lv]
    opts = ohm.default_opts(rtol=1e-8, precision=precision, max_iters=60)
    dt = (spec.dx0 / 2) ** 2 * 20.0
    got = []
    for n in (1, 8):
        b = [torch.cat([x] * n, dim=1) for x in B]
        e = [torch.cat([x] * n, dim=1) for x in E]
        st, stats = ohm.ohm_cn_step(ohm.Hierarchy([(spec.base_blocks, spec.dx0, lv)] * n), b, e, [dt] * n, opts)
        assert st == 0
        got.append(([x[:, :len(l)] for x, l in zip(b, lv)], stats[0]["iters"]))
    assert got[0][1] == got[1][1]
    for x, y in zip(got[0][0], got[1][0]):
        assert torch.equal(x, y)
