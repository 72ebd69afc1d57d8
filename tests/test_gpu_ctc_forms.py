"""The forms in which ctc_loss's recursions hold their values: doubles against the lanes' own exponents while every log2 p is at
least -60, mantissa and exponent below that.  Labels whose tokens are improbable in every frame, in little more frames than
labels (the values of a block of states spread furthest then) and in many, on both sides of the line; one frame across it."""
import math

import numpy as np
import pytest

from test_gpu_ctc_pipeline import _check, pkg  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("low", [-25.0, -36.0, -38.5, -39.5, -60.0])  # log2 p of the labels: -40 to -91, the line is at -60
@pytest.mark.parametrize("T,L", [(70, 66), (140, 135), (300, 130), (200, 20)])
def test_improbable_labels(pkg, T, L, low):  # noqa: F811
    rng = np.random.Generator(np.random.PCG64(T + L))
    B, C = 2, 13
    print(f"ctc_loss T={T} L={L} low={low}", flush=True)
    labels = np.tile(np.arange(L, dtype=np.int32) % 6, (B, 1))  # tokens 0 to 5; the others and the blank take the weight
    logits = rng.standard_normal((B, T, C), dtype=np.float32)
    logits[:, :, :6] += np.float32(low)
    # alpha and beta leave as float32 logarithms against the largest of 64 pairs of states, which spread over 64 x |log2 p|: an
    # occupancy is formed from four numbers of that size, each half an ulp off; an occupancy of up to one stands against an rms of
    # the gradient of at least a quarter (13 symbols, most rows with nearly all of their weight off by one entry)
    ulp = 2.0 ** (math.floor(math.log2(64 * (5 - low / math.log(2)))) - 23)
    tol = max(1e-4, 4 * 4 * ulp / 2 * math.log(2))
    _check(pkg, logits, labels, np.array([L, L - 3], dtype=np.int32), np.array([T, T - 1], dtype=np.int32), C - 1, tol)


@pytest.mark.parametrize("value", [-41.0, -43.0])  # log2 p of about -63 and -66
@pytest.mark.parametrize("frame", [0, 15, 16, 89])
def test_one_frame_across_the_line(pkg, value, frame):  # noqa: F811
    rng = np.random.Generator(np.random.PCG64(3))
    B, T, C, L = 2, 90, 23, 40
    logits = rng.standard_normal((B, T, C), dtype=np.float32)
    labels = np.tile(np.arange(L, dtype=np.int32) % 20, (B, 1))
    logits[0, frame, 3] = value
    _check(pkg, logits, labels, np.full(B, L, dtype=np.int32), np.full(B, T, dtype=np.int32), C - 1)
