"""GPU parity of weighted sums at the edges of their blocks and grids. Short first dimensions of the
direct form (sheared tilers), around the powers of two that its lanes take and the rest of a block's 256
points, with identity and permuted outputs. More blocks than one grid holds: the launch is cut, and every
piece computes its own blocks; |y - y64| <= 4 * 2^-24 * sum_i |w_i x_i| (three fused multiply-adds)."""

import numpy as np
import pytest

import synthgen

import torch

import paper_1103_4881_amd as aol  # a missing library fails the suite (no skip)
from tests.test_gpu_wsum_forms import _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fit", [[1, 0], [300, 7]])  # a box of a block's inputs, and none
def test_more_blocks_than_a_grid(fit):
    n, S = 2 ** 23 + 5, (1031, 1000)
    rep = (n, 2, 1)  # the loop dimension of a block is the last one, of one point: n blocks
    A = synthgen.rng_for(1, 2).uniform(-1, 1, size=S).astype(np.float32)
    w = np.array([0.5, -1.25, 0.75], np.float32)
    tin = aol.make_tiler(S, rep, (3,), (3, 4), [[7, 0, 0], [1, 1, 0]], [[fit[0]], [fit[1]]])
    plan = aol.WeightedSumPlan(tin, aol.identity_out_tiler(rep), w)
    x, y = torch.from_numpy(A).cuda(), torch.full(rep, float("nan"), dtype=torch.float32, device="cuda")
    plan.run(x, y)
    torch.cuda.synchronize()
    plan.close()
    r0, r1 = torch.arange(n, device="cuda")[:, None], torch.arange(2, device="cuda")[None]
    want = torch.zeros((n, 2), dtype=torch.float64, device="cuda")
    mag = torch.zeros_like(want)
    for i in range(3):
        v = float(w[i]) * x[(3 + 7 * r0 + fit[0] * i) % S[0], (4 + r0 + r1 + fit[1] * i) % S[1]].double()
        want += v
        mag += v.abs()
    assert ((y[:, :, 0].double() - want).abs() <= 4 * 2.0 ** -24 * mag).all()


@pytest.mark.parametrize("lane", [1, 2, 3, 4, 5, 8, 9, 16, 17, 32, 33])
@pytest.mark.parametrize("pat", [(3, 1), (2, 5)])
def test_direct_short_lanes(lane, pat):
    for loop in (1, 256 // lane - 1, 256 // lane + 1, 300):
        shape = (lane + 40, 2 * loop + 30, 3 * lane + 350)
        paving = [[1, 0, 9], [0, 2, 7], [0, 3, 1]]  # the lane dimension walks all three axes: no box fits
        for flip in (False, True):
            _case(shape, (3, loop, lane), pat, (5, 1, 2), paving, [[1, 0], [0, 0], [0, -50]], flip)
        _case((lane + 40, 2 * loop + 30), (loop, lane), pat, (5, 1), [[5, 1], [2, 1]], [[1, 0], [0, -50]])
