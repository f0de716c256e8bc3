"""The marching kernels where they do march (asserted from the plan): boxes one
tile across, with edges that are no multiple of the tiles and with short last
segments, and batches with problems of a block across, bit for bit against the
kernels per 8^3 block."""
import numpy as np
import pytest

import ohm_inputs as gen

from gpu_util import announce, cuda
from march_util import ALL, march_plan

pytestmark = pytest.mark.gpu


# one tile across in x and in y (its halo is the tile itself), odd edges; each
# with a last segment shorter than the others
@pytest.mark.parametrize("bb", [(2, 32, 57), (32, 2, 57), (13, 21, 19)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_marching_box_equals_blocks(bb, dtype):
    import torch
    import paper_1009_0798_amd as ohm
    announce(f"marching box == per block {bb} {dtype}")
    kernels, segs = march_plan([bb])
    assert kernels == ALL and len(set(segs[:, 5].tolist())) == 2
    tdt = torch.float64 if dtype == "f64" else torch.float32
    rng = np.random.default_rng(61)
    ijk = gen.full_level(bb)
    nb = len(ijk)
    B, S = (cuda(rng.standard_normal((3, nb, 8, 8, 8)), tdt) for _ in range(2))
    E = cuda(np.exp(rng.uniform(-2, 2, (1, nb, 8, 8, 8))), tdt)
    H = ohm.Hierarchy([(bb, 0.05, [ijk])])
    lam_dt = 0.05 ** 2 * 3.0
    # S off the pairs' alignment: the sweep per block
    off = torch.empty(S.numel() + 1, dtype=tdt, device="cuda")[1:].view(S.shape).copy_(S)
    assert off.data_ptr() % (2 * S.element_size()) != 0 and S.data_ptr() % (2 * S.element_size()) == 0
    got = []
    for s in (S, off):
        b = B.clone()
        ohm.ohm_smooth(H, 0, b, s, E, lam_dt, 3, torch.full_like(B, float("nan")))
        got.append(b)
    assert torch.equal(got[0], got[1]) and not torch.equal(got[0], B)
    # a residual with its norms is taken per block
    R, blk, out = (torch.full_like(B, float("nan")) for _ in range(3))
    ohm.ohm_residual(H, 0, B, S, E, lam_dt, R=blk, norms=True)
    ohm.ohm_residual(H, 0, B, S, E, lam_dt, R=R)
    assert torch.equal(R, blk)
    ohm.ohm_residual(H, 0, B, torch.zeros_like(S), E, lam_dt, R=blk, norms=True)
    ohm.ohm_apply(H, 0, B, E, lam_dt, out)
    assert torch.equal(out, -blk)


ODD = [(1, 1, 1), (1, 3, 5), (2, 1, 7), (3, 5, 4), (5, 2, 6), (2, 2, 3), (1, 6, 1), (6, 1, 2)]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("post", [3, 4])
def test_marching_batch_steps(precision, post):
    """Whole steps of a batch that marches (zero-guess sweeps, sweeps that add
    the coarse correction, sweeps with an FP64 result, the operator with its
    dot products, the residual with its restriction) and of its problems alone,
    which do not."""
    import torch
    import paper_1009_0798_amd as ohm
    announce(f"marching batch steps precision {precision} post {post}")
    boxes = ODD[:4] + [(4, 4, 4)] * 56 + ODD[4:]
    kernels, segs = march_plan(boxes)
    assert kernels == ALL and len(set(segs[:, 5].tolist())) == 2
    rng = np.random.default_rng(67)
    ijk = [gen.full_level(b) for b in boxes]
    dx = 0.05
    B = [rng.standard_normal((3, len(q), 8, 8, 8)) for q in ijk]
    E = [np.exp(rng.uniform(-1, 1, (1, len(q), 8, 8, 8))) for q in ijk]
    dts = [float(dx * dx * rng.uniform(3, 30)) for _ in boxes]
    opts = ohm.default_opts(rtol=1e-9, precision=precision, max_iters=80, nu_pre=2, nu_post=post, nu_coarse=1)
    both = cuda(np.concatenate(B, axis=1))
    st, stats = ohm.ohm_cn_step(ohm.Hierarchy([(b, dx, [q]) for b, q in zip(boxes, ijk)]), [both],
                                [cuda(np.concatenate(E, axis=1))], dts, opts)
    assert st == 0
    off = np.cumsum([0] + [len(q) for q in ijk])
    for i in list(range(8)) + list(range(len(boxes) - 5, len(boxes))):
        assert march_plan([boxes[i]])[0] == 0
        b = cuda(B[i])
        st, one = ohm.ohm_cn_step(ohm.Hierarchy([(boxes[i], dx, [ijk[i]])]), [b], [cuda(E[i])], dts[i], opts)
        assert st == 0 and one[0]["iters"] == stats[i]["iters"], i
        assert torch.equal(b, both[:, off[i]:off[i + 1]]), i
