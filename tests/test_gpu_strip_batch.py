"""GPU parity of batches on the strip kernel: streams of every filter class (K-steps of both axes, int8
and split taps) with lines of whole 16-byte chunks and others (two launches), shorter than a chunk, one
16-row block and many; short and long segments. Integer results are exact. Float results keep the bound
of their arithmetic: with |x| <= 1, A the largest sum of |c| / 256 over an axis' phases, products exact,
sums of at most 128 terms in float32 and the intermediate as two 16-bit halves,
|y - y64| <= Ah Av (2 * 130 * 2^-24 + 2^-16)."""

import json

import numpy as np
import pytest

import synthgen
from oracle import polyphase as pp

import torch

import paper_1103_4881_amd as aol  # a missing library fails the suite (no skip)

pytestmark = pytest.mark.gpu

WHOLE = [  # (h, w, p, q, taps, kind)
    (9, 16, 1, 2, 8, "design"), (96, 512, 1, 2, 8, "uneven"), (130, 704, 3, 8, 14, "design"),
    (70, 400, 3, 8, 16, "design"), (64, 384, 2, 3, 16, "design"), (70, 208, 16, 24, 9, "design"),
    (90, 256, 5, 7, 9, "uneven"), (200, 400, 1, 12, 30, "design"), (300, 304, 1, 5, 32, "uneven"),
    (640, 1296, 1, 2, 12, "design"),
]
EDGES = [
    (40, 5, 1, 2, 8, "design"), (98, 514, 1, 2, 8, "design"), (130, 701, 3, 8, 16, "design"),
    (66, 390, 2, 3, 16, "uneven"), (90, 261, 5, 7, 9, "design"), (300, 301, 1, 5, 32, "uneven"),
]


def _filter(p, q, taps, kind, seed):
    c = synthgen.design_taps(p, q, taps)
    if kind == "uneven":  # phases of different sums: biases that differ along an axis
        c = np.random.default_rng(seed).integers(-40, 60, c.shape).astype(np.int16)
    return aol.Polyphase(p, q, c), pp.Filter(p, q, c)


def _batch(shapes, fmt):
    filt = [(_filter(p, q, t, k, 2 * i), _filter(p, q, t, k, 2 * i + 1)) for i, (_, _, p, q, t, k) in enumerate(shapes)]
    plan = aol.BatchPlan([(s[0], s[1], hf[0], vf[0]) for s, (hf, vf) in zip(shapes, filt)], fmt)
    return plan, [(hf[1], vf[1]) for hf, vf in filt]


def _run(plan, ins, fill, dtype):
    outs = [torch.full(s, fill, dtype=dtype, device="cuda") for s in plan.out_shapes]
    plan.set_pointers(ins, outs)
    plan.run()
    torch.cuda.synchronize()
    return [o.cpu().numpy() for o in outs]


@pytest.mark.parametrize("shapes,launches", [(WHOLE, 1), (EDGES, 1), (WHOLE + EDGES, 2)],
                         ids=["whole", "edges", "mixed"])
def test_integer_batch(shapes, launches):
    plan, filt = _batch(shapes, "u8")
    assert json.loads(plan.schedule())["launches"] == launches
    frames = [synthgen.uniform_frame(i, s[0], s[1], idx=i) for i, s in enumerate(shapes)]
    want = [pp.downscale_u8(f, hf, vf) for f, (hf, vf) in zip(frames, filt)]
    ins = [torch.from_numpy(f).cuda() for f in frames]
    for k, seg in enumerate((None, 16, 128)):
        if seg:
            plan.set_schedule(seg, 150 * 1024)
        for i, y in enumerate(_run(plan, ins, 0xFF if k % 2 else 0x00, torch.uint8)):
            np.testing.assert_array_equal(y, want[i], err_msg=f"segments {seg}: stream {i} {shapes[i]}")
    plan.close()


@pytest.mark.parametrize("fmt", ["bf16", "fp16"])
def test_float_batch(fmt):
    shapes = [s[:5] + ("design",) for s in WHOLE + EDGES if s[4] <= 16]
    plan, filt = _batch(shapes, fmt)
    bits = [synthgen.normalised(synthgen.uniform_frame(i, s[0], s[1], idx=i), fmt) for i, s in enumerate(shapes)]
    ins = [torch.from_numpy(b.view(np.int16)).cuda() for b in bits]
    for seg in (None, 16):
        if seg:
            plan.set_schedule(seg, 150 * 1024)
        for i, y in enumerate(_run(plan, ins, float("nan"), torch.float32)):
            x = (bits[i].astype(np.uint32) << 16).view(np.float32) if fmt == "bf16" else bits[i].view(np.float16)
            amp = np.abs(synthgen.design_taps(*shapes[i][2:5]).astype(np.float64)).sum(axis=1).max() / 256
            err = np.abs(y - pp.downscale_f64(x.astype(np.float64), *filt[i])).max()
            assert err <= amp * amp * (260 * 2.0 ** -24 + 2.0 ** -16), f"segments {seg}: stream {i} {shapes[i]}"
    plan.close()
