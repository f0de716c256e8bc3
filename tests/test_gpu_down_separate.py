"""The way down from a dense level in one launch (sweep from zero, residual,
restriction, on parts of the tiles) against the separate kernels of whole tiles,
bit for bit.  A 64 x 8 x 8 box in the handle, whose coarsest grid has an edge of
2 cells at the second dense level, sends that level of every problem to the
separate kernels."""
import numpy as np
import pytest

import ohm_inputs as gen

from gpu_util import announce, cuda

pytestmark = pytest.mark.gpu


# problems of 48^3 cells: the second dense level has 8 tiles, which overhang its
# 12^3 cells, of each: 8 (quarters), 96 (halves), and 320 (FP32 only: halves)
@pytest.mark.parametrize("precision,count", [(0, 1), (0, 12), (1, 1), (1, 12), (1, 40)])
def test_fused_equals_separate(precision, count):
    import torch
    import paper_1009_0798_amd as ohm
    announce(f"way down fused == separate precision {precision} x {count}")
    rng = np.random.default_rng(73)
    boxes = [(6, 6, 6)] * count + [(8, 1, 1)]
    ijk = [gen.full_level(b) for b in boxes]
    B = [rng.standard_normal((3, len(q), 8, 8, 8)) for q in ijk]
    E = [np.exp(rng.uniform(-1, 1, (1, len(q), 8, 8, 8))) for q in ijk]
    dx, dt = 0.05, 0.05 ** 2 * 30.0
    opts = ohm.default_opts(rtol=1e-9, precision=precision, max_iters=60, nu_pre=2, nu_post=3, nu_coarse=1)
    got = []
    for n in (count, count + 1):
        b = cuda(np.concatenate(B[:n], axis=1))
        H = ohm.Hierarchy([(bb, dx, [q]) for bb, q in zip(boxes[:n], ijk[:n])])
        assert H.problem_info(0, -2)[1] == (12, 12, 12) and H.prob_min_level[0] < -2
        st, stats = ohm.ohm_cn_step(H, [b], [cuda(np.concatenate(E[:n], axis=1))], [dt] * n, opts)
        assert st == 0
        got.append((b, [s["iters"] for s in stats]))
    assert H.problem_info(count, -2)[1] == (16, 2, 2) and H.prob_min_level[count] == -2
    nb = got[0][0].shape[1]
    assert got[0][1] == got[1][1][:count] and torch.equal(got[0][0], got[1][0][:, :nb])
