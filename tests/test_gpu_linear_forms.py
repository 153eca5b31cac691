"""GPU parity of the linear integer repetition's packed and matrix-core forms against the CPU oracle,
bit-exact, at the sizes where they can go wrong: runs around 16 points of a thread and 4,096 of a
workgroup, components in any order, rows that do not continue each other; blocks of 32 x 8 points and
one off, axes shorter than a 16-byte chunk, patterns that wrap on every side, chunk positions of every
alignment, negative pavings, weights of one and of two int8 parts and beyond them, two elements on one
position. Each case runs on aligned arrays and on views one byte off, over two sentinel fills."""

import numpy as np
import pytest

import synthgen
from tests.test_gpu_linear import _frames_spec, _oracle, _run

pytestmark = pytest.mark.gpu

SPEC = synthgen.TilerSpec


@pytest.mark.parametrize("h,w", [(1, 1), (1, 15), (1, 16), (3, 17), (5, 819), (64, 64), (2, 4097)])
@pytest.mark.parametrize("n", [1, 3])
def test_colour_conversions(h, w, n):
    X = synthgen.uniform_frame(h + w, n * h, 3 * w).reshape(n, h, 3 * w)
    rep, ti, to = synthgen.rgb_to_planar_tilers(h, w)
    ti, to = _frames_spec(ti, n), _frames_spec(to, n)
    Y = _run(X, ti, to, (n,) + rep, synthgen.RGB_TO_YCC_W, synthgen.RGB_TO_YCC_BIAS)
    np.testing.assert_array_equal(Y, _oracle(X, ti, to, (n,) + rep, synthgen.RGB_TO_YCC_W, synthgen.RGB_TO_YCC_BIAS))
    rep, ti, to = synthgen.planar_to_rgb_tilers(h, w)
    ti, to = _frames_spec(ti, n), _frames_spec(to, n)
    Z = _run(Y, ti, to, (n,) + rep, synthgen.YCC_TO_RGB_W, synthgen.YCC_TO_RGB_BIAS)
    np.testing.assert_array_equal(Z, _oracle(Y, ti, to, (n,) + rep, synthgen.YCC_TO_RGB_W, synthgen.YCC_TO_RGB_BIAS))


@pytest.mark.parametrize("origin,step", [(0, 1), (2, -1)])
@pytest.mark.parametrize("pad", [0, 5])
def test_component_order_padding_and_large_weights(origin, step, pad):
    """Components from the last to the first (a negative fitting), input rows with unused bytes at
    their end (the rows' points are no longer one run), planes in reverse order, weights to +-32767."""
    h, w = 9, 37
    X = synthgen.uniform_frame(7, h, 3 * w + pad)
    W = np.array([[32767, -32768, 5], [256, 0, 0], [-3, 700, 300]], np.int32).astype(np.int16)
    tin = SPEC((h, 3 * w + pad), (0, origin), [[1, 0], [0, 3]], [[0], [step]], (3,))
    tout = SPEC((3, h, w), (2, 0, 0), [[0, 0], [1, 0], [0, 1]], [[-1], [0], [0]], (3,))
    bias = np.array([-70000, 3, 90000], np.int32)
    np.testing.assert_array_equal(_run(X, tin, tout, (h, w), W, bias), _oracle(X, tin, tout, (h, w), W, bias))


# (h, w, p, q, taps, weight scale)
@pytest.mark.parametrize("case", [(12, 13, 1, 2, 8, 1), (40, 64, 1, 2, 8, 1), (34, 66, 1, 2, 9, 3), (64, 256, 3, 8, 11, 1),
                                  (72, 264, 3, 8, 11, 4), (50, 99, 2, 3, 9, 1), (33, 96, 2, 3, 12, 2), (70, 71, 3, 8, 8, 200)],
                         ids=str)
def test_windows(case):
    h, w, p, q, taps, scale = case
    n = 2
    X = synthgen.uniform_frame(h * 3 + w, n * h, w).reshape(n, h, w)
    rep, ti, to, _, _ = synthgen.polyphase2d_tilers(h, w, p, q, taps)
    W = (synthgen.polyphase2d_weights(5, p, q, taps).astype(np.int32) * scale).clip(-32768, 32767).astype(np.int16)
    ti, to = _frames_spec(ti, n), _frames_spec(to, n)
    np.testing.assert_array_equal(_run(X, ti, to, (n,) + rep, W, None), _oracle(X, ti, to, (n,) + rep, W, None))


@pytest.mark.parametrize("fit", [[[1, 0], [0, 1]], [[0, -2], [3, 0]], [[1, 1], [0, 0]]])
def test_negative_pavings_strided_and_coinciding_elements(fit):
    """A 6 x 7 pattern read backwards along both axes, with strides, transposed, or with several
    elements on one position; outputs in reverse."""
    h, w = 41, 70
    X = synthgen.uniform_frame(11, h, w)
    g = synthgen.rng_for(3, 1)
    W = g.integers(-128, 128, size=(1, 42)).astype(np.int16)
    tin = SPEC((h, w), (3, 5), [[-1, 0], [0, -1]], fit, (6, 7))
    tout = SPEC((h, w), (h - 1, w - 1), [[-1, 0], [0, -1]], [[], []], ())
    np.testing.assert_array_equal(_run(X, tin, tout, (h, w), W, None), _oracle(X, tin, tout, (h, w), W, None))


def test_one_repetition_dimension():
    X = synthgen.uniform_frame(12, 1, 300).reshape(300)
    W = synthgen.rng_for(3, 2).integers(-300, 300, size=(2, 40)).astype(np.int16)
    tin = SPEC((300,), (290,), [[2]], [[3]], (40,))
    tout = SPEC((300,), (0,), [[2]], [[1]], (2,))
    np.testing.assert_array_equal(_run(X, tin, tout, (150,), W, None), _oracle(X, tin, tout, (150,), W, None))
