"""Infinities and NaN in float frames, on the strip kernel: every output whose taps reach one is not
finite, and no output of a 16 x 16 block whose window does not hold it is touched: the block's own lines,
and its own columns to the 8-element chunks that hold them. Whatever the schedule: plans' segments, one
frame and so many that the eight-wave form runs, batches."""

import numpy as np
import pytest

import synthgen

import torch

import paper_1103_4881_amd as aol  # a missing library fails the suite (no skip)
from oracle import polyphase as pp

pytestmark = pytest.mark.gpu

DT = {"bf16": torch.bfloat16, "fp16": torch.float16}


def _reach(f, n, size, at, chunk):
    """(outputs of one axis whose taps hold element `at`, 16-output blocks whose window, widened to
    multiples of `chunk`, holds it), as masks over the n outputs."""
    hit, blocks = np.zeros(n, bool), np.zeros(n, bool)
    first = [f.q * (o // f.p) + f.s[o % f.p] for o in range((n + 15) // 16 * 16)]
    for o in range(n):
        hit[o] = any((first[o] + k) % size == at and f.c[o % f.p][k] != 0 for k in range(f.T))
    for b in range(0, n, 16):
        lo = min(first[b:b + 16]) // chunk * chunk
        hi = -(-(max(first[b:b + 16]) + f.T) // chunk) * chunk
        blocks[b:b + 16] = any((x - at) % size == 0 for x in range(lo, hi))
    return hit, blocks


def _check(bad, of, shape, points):
    want, may = np.zeros(bad.shape, bool), np.zeros(bad.shape, bool)
    for y, x in points:
        (hy, by), (hx, bx) = _reach(of, bad.shape[0], shape[0], y, 1), _reach(of, bad.shape[1], shape[1], x, 8)
        want |= hy[:, None] & hx[None]
        may |= by[:, None] & bx[None]
    assert bad[want].all(), "an output over a NaN is finite"
    assert not bad[~may].any(), "an output of a block that holds no NaN is not finite"


FILTERS = [(1, 2, 8), (2, 3, 8), (5, 7, 9), (3, 8, 11), (1, 5, 12), (3, 8, 16), (1, 7, 14)]


@pytest.mark.parametrize("fmt", ["bf16", "fp16"])
@pytest.mark.parametrize("p,q,taps", FILTERS)
@pytest.mark.parametrize("shape", [(320, 336), (331, 341)])
def test_plans(fmt, p, q, taps, shape):
    c = synthgen.design_taps(p, q, taps)
    f, of = aol.Polyphase(p, q, c), pp.Filter(p, q, c)
    points = [(0, 0), (shape[0] - 1, 170), (151, shape[1] - 1), (160, 90), (175, 203), (96, 16)]
    first = None
    for n in (1, 300):
        x = torch.rand((n,) + shape, device="cuda").to(DT[fmt])
        x[0] = torch.rand(shape, device="cuda", generator=torch.Generator("cuda").manual_seed(1)).to(DT[fmt])
        for i, (r, col) in enumerate(points):
            x[0, r, col] = float("nan") if i % 2 else float("inf")
        for seg in (0, 16, 48, 64):
            plan = aol.DownscalePlan([shape], f, f, fmt)
            if seg:
                plan.set_band(0, seg)
            y = torch.zeros((n,) + plan.out_shapes[0], device="cuda")
            plan.run([x], [y])
            torch.cuda.synchronize()
            plan.close()
            got = y[0].cpu().numpy()
            _check(~np.isfinite(got), of, shape, points)
            first = got if first is None else first
            np.testing.assert_array_equal(got, first, err_msg=f"{n} frames, segments of {seg}")
            assert n == 1 or bool(torch.isfinite(y[1:]).all())


@pytest.mark.parametrize("fmt", ["bf16", "fp16"])
def test_batch(fmt):
    shapes = [(320, 336), (331, 341)]
    filt = [synthgen.design_taps(*f) for f in FILTERS]
    streams = [(s, aol.Polyphase(p, q, c), pp.Filter(p, q, c)) for s in shapes for (p, q, _), c in zip(FILTERS, filt)]
    plan = aol.BatchPlan([(s[0], s[1], f, f) for s, f, _ in streams], fmt)
    ins, points = [], [(151, 7), (160, 90), (9, 203)]
    for i, (s, _, _) in enumerate(streams):
        x = torch.rand(s, device="cuda", generator=torch.Generator("cuda").manual_seed(i)).to(DT[fmt])
        for r, col in points:
            x[r, col] = float("nan")
        ins.append(x)
    first = None
    for seg in (0, 16, 64):
        plan.set_schedule(seg, 150 * 1024)
        outs = [torch.zeros(s, device="cuda") for s in plan.out_shapes]
        plan.set_pointers(ins, outs)
        plan.run()
        torch.cuda.synchronize()
        got = [o.cpu().numpy() for o in outs]
        for y, (s, _, of) in zip(got, streams):
            _check(~np.isfinite(y), of, s, points)
        first = got if first is None else first
        for a, b in zip(got, first):
            np.testing.assert_array_equal(a, b, err_msg=f"segments of {seg}")
    plan.close()
