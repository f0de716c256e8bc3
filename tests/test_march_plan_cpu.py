"""The plan of the marching kernels (plain host code): every block of every
problem in one segment, segments within the kernels' limits, the XCDs' runs of
about equal work, and no plan for base levels of few blocks."""
import numpy as np
import pytest

from march_util import ALL, FP32_SWEEPS, FP64_RESIDUAL, FP64_SWEEPS, OPERATOR, march_plan


def _check(boxes):
    kernels, segs = march_plan(boxes)
    assert (kernels == 0) == (len(segs) == 0)
    if not kernels:
        return False
    cover = [np.zeros(b, dtype=int) for b in boxes]
    for x, p, i, j, k, n in segs:
        assert i % 2 == 0 and j % 2 == 0 and 1 <= n <= 32 and k + n <= boxes[p][2]
        cover[p][i:i + 2, j:j + 2, k:k + n] += 1
    for c in cover:
        assert (c == 1).all()
    assert (np.diff(segs[:, 0]) >= 0).all() and segs[0, 0] >= 0 and segs[-1, 0] <= 7
    # a column's planes and as many again as one block's to start: no XCD has
    # more than one segment over an eighth
    work = np.zeros(8)
    np.add.at(work, segs[:, 0], 8 * segs[:, 5] + 8)
    assert work.max() <= work.sum() / 8 + 8 * segs[:, 5].max() + 8
    return True


@pytest.mark.parametrize("boxes", [[(16, 16, 16)], [(17, 13, 21)], [(2, 32, 57)], [(32, 2, 57)], [(27, 32, 6)],
                                   [(2, 2, 1100)], [(32, 32, 32)], [(4, 4, 4)] * 64,
                                   [(4, 4, 4)] * 56 + [(1, 1, 1), (1, 3, 5), (2, 1, 7), (3, 5, 4), (5, 2, 6)]])
def test_every_block_in_one_segment(boxes):
    assert _check(boxes)


def test_random_handles():
    rng = np.random.default_rng(3)
    marching = 0
    for _ in range(150):
        if rng.random() < 0.5:
            boxes = [tuple(int(v) for v in rng.integers(1, 40, 3))]
        else:
            boxes = [tuple(int(v) for v in rng.integers(1, 9, 3)) for _ in range(int(rng.integers(2, 120)))]
        marching += _check(boxes)
    assert marching > 20


# sizes on either side of each kernel's line; those without a kernel were timed
# and the kernel per block is the faster one there
@pytest.mark.parametrize("boxes,kernels", [
    ([(1, 1, 1)], 0), ([(8, 8, 8)], 0), ([(14, 14, 14)], 0), ([(4, 4, 4)] * 32, 0), ([(1, 64, 64)], 0),
    ([(16, 16, 16)], ALL), ([(20, 16, 24)], ALL), ([(24, 24, 24)], ALL), ([(4, 4, 4)] * 64, ALL), ([(32, 32, 21)], ALL),
    ([(19, 19, 19)], ALL - FP32_SWEEPS), ([(22, 22, 22)], ALL - FP32_SWEEPS),
    ([(21, 21, 21)], ALL - FP32_SWEEPS), ([(27, 33, 12)], ALL),
    ([(23, 40, 5)], OPERATOR + FP64_RESIDUAL), ([(27, 33, 7)], ALL - FP32_SWEEPS),
    ([(4, 4, 4)] * 96, ALL - FP64_RESIDUAL), ([(25, 18, 15)], ALL - FP32_SWEEPS), ([(4, 4, 4)] * 159, ALL),
    ([(12, 12, 12)] * 3, ALL)])
def test_what_marches(boxes, kernels):
    assert march_plan(boxes)[0] == kernels
