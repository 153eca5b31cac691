"""GPU parity of the linear integer repetition on an axis close to 2^31 elements, where the sum of two
coordinates passes 2^31: windows that wrap at the end of the axis, offsets of more than half of it,
steps of a point's successor that wrap (rows of more than one point per thread). The wanted sums are
taken element by element in int64 from the same array."""

import numpy as np
import pytest

import synthgen

import torch

import paper_1103_4881_amd as aol  # a missing library fails the suite (no skip)

pytestmark = pytest.mark.gpu

S = 2 ** 31 - 77


@pytest.fixture(scope="module")
def axis():
    x = torch.empty(S, dtype=torch.uint8, device="cuda")
    for k in range(0, S, 1 << 28):  # every byte of its low and high neighbourhood different
        part = torch.arange(k, min(S, k + (1 << 28)), device="cuda", dtype=torch.int64)
        x[k:k + len(part)] = ((part * 40503) >> 7).to(torch.uint8)
    yield x
    del x
    torch.cuda.empty_cache()


# (origin, paving of the rows, paving along a row, fitting, pattern elements)
@pytest.mark.parametrize("case", [(S - 100, 7, 3, 1, 40), (S - 5, -1, S - 7, -3, 50), (5, 1 << 30, 1, 700_000_003, 3),
                                  (S // 2, 3, 1_500_000_001, 1_000_000_007, 4), (S - 1, 0, 1, 1, 33)], ids=str)
def test_axis_close_to_2_31(axis, case):
    o, prow, plast, fit, k = case
    rep = (16, 700)
    W = synthgen.rng_for(k, 1).integers(-100, 128, size=(2, k)).astype(np.int16)
    plan = aol.LinearPlan(aol.make_tiler((S,), rep, (k,), (o,), [[prow, plast]], [[fit]]),
                          aol.make_tiler(rep + (2,), rep, (2,), (0, 0, 0), [[1, 0], [0, 1], [0, 0]], [[0], [0], [1]]), W)
    y = torch.full(rep + (2,), 0xA5, dtype=torch.uint8, device="cuda")
    plan.run(axis, y)
    torch.cuda.synchronize()
    plan.close()
    r0, r1, i = np.ogrid[:rep[0], :rep[1], :k]
    at = (o + prow * r0 + plast * r1 + fit * i) % S  # Python's modulus: below S
    v = axis[torch.from_numpy(at.astype(np.int64)).cuda()].cpu().numpy().astype(np.int64)
    want = np.clip((v @ W.astype(np.int64).T + 128) >> 8, 0, 255)
    np.testing.assert_array_equal(y.cpu().numpy(), want)
