"""GPU parity of the weighted sum's two forms at the sizes where they can go wrong: staged boxes whose
rows are whole 16-byte chunks, one element off, shorter than a chunk and wrapped several times; the
direct form (sheared tilers) with 1 to 64 pattern elements, around its groups of eight, and repetition
spaces around its blocks of 64 x 4 points, with identity and permuted outputs. |y - y64| <= 64 * 2^-24 *
sum_i |w_i x_i| (at most 64 fused multiply-adds in float32)."""

import numpy as np
import pytest

import synthgen
from oracle import generic as gn
from oracle.arrayol import Tiler

import torch

import paper_1103_4881_amd as aol  # a missing library fails the suite (no skip)

pytestmark = pytest.mark.gpu


def _case(shape, rep, pat, origin, paving, fitting, flip=False):
    A = synthgen.rng_for(sum(shape), 1).uniform(-1, 1, size=shape).astype(np.float32)
    w = synthgen.rng_for(sum(pat), 2).uniform(-1, 1, size=pat).astype(np.float32)
    tin = aol.make_tiler(shape, rep, pat, origin, paving, fitting)
    if flip:  # output axes reversed
        n = len(rep)
        oshape, opaving = tuple(reversed(rep)), [[1 if d == n - 1 - k else 0 for k in range(n)] for d in range(n)]
    else:
        oshape, opaving = rep, np.eye(len(rep), dtype=int).tolist()
    tout = aol.make_tiler(oshape, rep, (1,), (0,) * len(rep), opaving, [[0]] * len(rep))
    plan = aol.WeightedSumPlan(tin, tout, w)
    y = torch.full(plan.out_shape, float("nan"), dtype=torch.float32, device="cuda")
    plan.run(torch.from_numpy(A).cuda(), y)
    torch.cuda.synchronize()
    plan.close()
    ot = Tiler(shape, origin, paving, fitting, pat)
    oo = Tiler(oshape, (0,) * len(rep), opaving, [[0]] * len(rep), (1,))
    B, M, _ = gn.weighted_sum_f64(A, ot, w, oo, rep)
    assert (np.abs(y.cpu().numpy().astype(np.float64) - B) <= 64 * 2.0 ** -24 * np.maximum(M, 1e-30)).all()


@pytest.mark.parametrize("w", [3, 5, 8, 63, 64, 65, 127, 130, 200])
@pytest.mark.parametrize("step,k", [(1, 2), (1, 5), (2, 3)])
def test_staged_rows(w, step, k):
    h = 37
    for origin in ((0, 0), (h - 1, w - 1)):
        _case((h, w), (h, -(-w // step)), (3, k), origin, [[1, 0], [0, step]], [[1, 0], [0, -1]])


@pytest.mark.parametrize("n", [33, 45, 48])
def test_staged_narrow_blocks(n):
    """Boxes that fit with 16 points of the second dimension a block, not with 32."""
    for flip in (False, True):
        _case((6, 2 * n, 201), (6, n, 101), (3, 1), (5, 2 * n - 3, 7), [[1, 0, 0], [0, 2, 0], [0, 0, 2]],
              [[1, 0], [0, 0], [0, 0]], flip)


@pytest.mark.parametrize("pat", [(1, 1), (7, 1), (2, 4), (3, 3), (3, 5), (4, 4), (8, 8)])
@pytest.mark.parametrize("rep", [(3, 64, 4), (5, 65, 5), (2, 63, 3), (1, 130, 9)])
def test_direct_sheared(pat, rep):
    shape = (rep[2] + 40, 2 * rep[1] + 3, rep[0] + 150)
    # the second dimension walks all three axes: no box of a block fits
    paving = [[0, 7, 1], [0, 2, 0], [1, 3, 0]]
    for flip in (False, True):
        _case(shape, rep, pat, (5, 1, 2), paving, [[1, 0], [0, 0], [0, -2]], flip)
