"""GPU parity of the strip kernel (the fused downscaler's default) at the sizes where it can go wrong:
lines shorter than a 16-byte chunk, of whole chunks and one off; output widths around 16-column
strips and a workgroup's 256 columns; output heights around 16-row blocks and segments; rows and
buffers at odd addresses; every class of filter (K-steps of both axes, int8 and split taps); launches
of one frame and of so many that the eight-wave form runs. Integer results are exact. Float results
keep the bound of their arithmetic: with |x| <= 1, A the largest sum of |c| / 256 over an axis' phases,
products exact, sums of at most 128 terms in float32 and the intermediate as two 16-bit halves,
|y - y64| <= Ah Av (2 * 130 * 2^-24 + 2^-16)."""

import numpy as np
import pytest

import synthgen
from oracle import polyphase as pp

import torch

import paper_1103_4881_amd as aol  # a missing library fails the suite (no skip)

pytestmark = pytest.mark.gpu


def _filter(p, q, taps, kind="design", seed=0):
    c = synthgen.design_taps(p, q, taps)
    if kind == "uneven":  # phases of different sums: biases that differ along an axis
        c = np.random.default_rng(seed).integers(-40, 60, c.shape).astype(np.int16)
    return aol.Polyphase(p, q, c), pp.Filter(p, q, c)


def _run(X, hf, vf, fmt="u8", off=0, pad=0):
    """Frames X [n, h, w] (bits for float forms) at `off` elements into their buffers, rows `pad`
    elements apart beyond the width; guard elements around the output must stay untouched."""
    n, h, w = X.shape
    plan = aol.DownscalePlan([(h, w)], hf, vf, fmt, in_pitches=[w + pad])
    oh, ow = plan.out_shapes[0]
    xb = torch.zeros(off + n * h * (w + pad) + 16, dtype=torch.uint8 if fmt == "u8" else torch.int16, device="cuda")
    x = xb[off:off + n * h * (w + pad)].view(n, h, w + pad)[:, :, :w]
    x.copy_(torch.from_numpy(X if fmt == "u8" else X.view(np.int16)))
    outs = []
    for fill in (0x11, 0xEE):
        yb = torch.full((off + n * oh * ow + 64,), fill, dtype=torch.uint8 if fmt == "u8" else torch.float32,
                        device="cuda")
        y = yb[off:off + n * oh * ow].view(n, oh, ow)
        plan.run([x], [y])
        torch.cuda.synchronize()
        assert (yb[:off] == fill).all() and (yb[off + n * oh * ow:] == fill).all(), "write outside the output"
        outs.append(y.cpu().numpy())
    plan.close()
    np.testing.assert_array_equal(outs[0], outs[1], err_msg="an output was not written")
    return outs[0]


# (h, w, p, q, taps, kind)
SHAPES = [
    (40, 5, 1, 2, 8, "design"), (40, 15, 3, 8, 11, "design"), (40, 16, 3, 8, 11, "design"),
    (40, 17, 3, 8, 11, "design"), (9, 31, 2, 3, 14, "design"),                 # short lines and columns
    (96, 512, 1, 2, 8, "design"), (98, 514, 1, 2, 8, "design"), (94, 510, 1, 2, 8, "uneven"),  # 256 columns, 48 rows
    (130, 701, 3, 8, 16, "design"), (130, 704, 3, 8, 14, "design"),            # two K-steps
    (66, 390, 2, 3, 16, "design"), (64, 385, 2, 3, 9, "uneven"),               # split taps, one workgroup and more
    (70, 200, 16, 24, 9, "design"), (90, 260, 5, 7, 9, "uneven"), (50, 150, 5, 3, 9, "design"),
    (200, 400, 1, 12, 30, "design"), (300, 300, 1, 5, 32, "uneven"),           # wide windows
]


@pytest.mark.parametrize("case", SHAPES, ids=["x".join(map(str, c)) for c in SHAPES])
@pytest.mark.parametrize("off,pad", [(0, 0), (1, 3)])
def test_integer_edges(case, off, pad):
    h, w, p, q, taps, kind = case
    hf, of = _filter(p, q, taps, kind, 1)
    vf, ov = _filter(p, q, taps, kind, 2)
    X = np.stack([synthgen.uniform_frame(h + f, h, w, idx=w) for f in range(2)])
    np.testing.assert_array_equal(_run(X, hf, vf, off=off, pad=pad), pp.downscale_u8(X, of, ov))


@pytest.mark.parametrize("fmt", ["bf16", "fp16"])
@pytest.mark.parametrize("case", [(40, 7, 1, 2, 8), (66, 390, 2, 3, 16), (130, 704, 3, 8, 16), (98, 514, 1, 2, 12),
                                  (70, 201, 3, 8, 11), (200, 300, 1, 5, 15)])
def test_float_edges(fmt, case):
    h, w, p, q, taps = case
    hf, of = _filter(p, q, taps)
    bits = synthgen.normalised(synthgen.uniform_frame(h, h, w)[None], fmt)
    x = (bits.astype(np.uint32) << 16).view(np.float32) if fmt == "bf16" else bits.view(np.float16)
    amp = np.abs(synthgen.design_taps(p, q, taps).astype(np.float64)).sum(axis=1).max() / 256
    for off, pad in [(0, 0), (1, 1)]:
        y = _run(bits, hf, hf, fmt, off=off, pad=pad)
        assert np.abs(y - pp.downscale_f64(x.astype(np.float64), of, of)).max() <= amp * amp * (
            260 * 2.0 ** -24 + 2.0 ** -16)


@pytest.mark.parametrize("fmt,w", [("u8", 64), ("bf16", 64), ("u8", 63)])
def test_many_frames(fmt, w):
    """2,500 frames: the eight-wave form where lines are whole chunks."""
    hf, of = _filter(3, 8, 11)
    U = np.stack([synthgen.uniform_frame(f, 40, w) for f in range(50)]).repeat(50, axis=0)
    U[::7] = 255 - U[::7]
    if fmt == "u8":
        np.testing.assert_array_equal(_run(U, hf, hf), pp.downscale_u8(U, of, of))
        return
    bits = synthgen.normalised(U, fmt)
    x = (bits.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    amp = np.abs(synthgen.design_taps(3, 8, 11).astype(np.float64)).sum(axis=1).max() / 256
    assert np.abs(_run(bits, hf, hf, fmt) - pp.downscale_f64(x, of, of)).max() <= amp * amp * (
        260 * 2.0 ** -24 + 2.0 ** -16)
