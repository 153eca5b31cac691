"""Float results are the same bits in every schedule, on every class of filter: segments of any length,
one frame and so many that the eight-wave form runs, plans and batches, lines of whole 16-byte chunks and
others."""

import numpy as np
import pytest

import synthgen

import torch

import paper_1103_4881_amd as aol  # a missing library fails the suite (no skip)

pytestmark = pytest.mark.gpu

DT = {"bf16": torch.bfloat16, "fp16": torch.float16}
FILTERS = [(1, 2, 8), (2, 3, 8), (5, 7, 9), (3, 8, 11), (1, 5, 12), (3, 8, 16), (1, 7, 14), (16, 24, 9), (5, 3, 6)]
SHAPES = [(320, 336), (331, 341)]


def _frames(shape, fmt, n=1):
    x = torch.rand((1,) + shape, device="cuda", generator=torch.Generator("cuda").manual_seed(shape[1]))
    return x.to(DT[fmt]).repeat(n, 1, 1)


@pytest.mark.parametrize("fmt", ["bf16", "fp16"])
@pytest.mark.parametrize("p,q,taps", FILTERS)
def test_float_results_do_not_depend_on_the_schedule(fmt, p, q, taps):
    f = aol.Polyphase(p, q, synthgen.design_taps(p, q, taps))
    batch = aol.BatchPlan([s + (f, f) for s in SHAPES], fmt)
    for i, shape in enumerate(SHAPES):
        got = []
        for n, seg in ((1, 0), (1, 16), (1, 32), (1, 48), (2, 64), (9, 0), (300, 0)):
            plan = aol.DownscalePlan([shape], f, f, fmt)
            if seg:
                plan.set_band(0, seg)
            y = torch.zeros((n,) + plan.out_shapes[0], device="cuda")
            plan.run([_frames(shape, fmt, n)], [y])
            torch.cuda.synchronize()
            plan.close()
            assert (y == y[:1]).all(), f"frames of one launch differ ({n} frames, segments of {seg})"
            got.append((f"{n} frames, segments of {seg}", y[0].cpu().numpy()))
        for seg in (0, 16, 48):
            batch.set_schedule(seg, 150 * 1024)
            outs = [torch.zeros(s, device="cuda") for s in batch.out_shapes]
            batch.set_pointers([_frames(s, fmt)[0] for s in SHAPES], outs)
            batch.run()
            torch.cuda.synchronize()
            got.append((f"batch, segments of {seg}", outs[i].cpu().numpy()))
        for name, y in got[1:]:
            np.testing.assert_array_equal(y, got[0][1], err_msg=f"{shape}: {name}")
    batch.close()
