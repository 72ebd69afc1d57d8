"""The forms in which ctc_loss's recursions hold their values: doubles against the states' own scales while every log2 p is at
least -40 and the values of neighbouring states allow for it, mantissa and exponent otherwise.  Labels whose tokens are improbable
in every frame, in little more frames than labels (the values of a block of states spread furthest then) and in many, on both sides of
the line; one frame across it; and states that count although they lie far behind, or far ahead of, those beside them."""
import math

import numpy as np
import pytest
import torch

import oracle
from test_gpu_ctc_pipeline import _check, pkg  # noqa: F401
from workloads.device import dev_f32, dev_i32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("low", [-20.0, -24.0, -25.0, -36.0, -38.5, -39.5, -60.0])  # log2 p of the labels: -33 to -91, the line is at -40
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


@pytest.mark.parametrize("value", [-23.0, -25.0, -41.0, -43.0])  # log2 p of about -38, -41, -63 and -66
@pytest.mark.parametrize("frame", [0, 15, 16, 89])
def test_one_frame_across_the_line(pkg, value, frame):  # noqa: F811
    rng = np.random.Generator(np.random.PCG64(3))
    B, T, C, L = 2, 90, 23, 40
    logits = rng.standard_normal((B, T, C), dtype=np.float32)
    labels = np.tile(np.arange(L, dtype=np.int32) % 20, (B, 1))
    logits[0, frame, 3] = value
    _check(pkg, logits, labels, np.full(B, L, dtype=np.int32), np.full(B, T, dtype=np.int32), C - 1)


# ---- states that lie far behind, and far ahead of, those beside them ---------------------------------------------------
def _far(pkg, logits, labels, copies, blank):  # noqa: F811
    """Sequences of full length; `copies` of the batch (many: the form with two writers, mantissas throughout)."""
    B, T, C = logits.shape
    L = labels.shape[1]
    # what counts in an occupancy is at least P: it lies at most -log2 P below the largest state of its block, and is formed from four
    # float32 numbers of that size, each half an ulp off, against an rms of the gradient of at least a quarter of an entry
    spread = max(oracle.ctc_loss_and_grad(logits[b], tuple(int(v) for v in labels[b]), blank)[0] for b in range(B)) / math.log(2)
    assert spread < math.inf
    tol = max(1e-4, 4 * 4 * 2.0 ** (math.floor(math.log2(spread + 1)) - 23) / 2 * math.log(2))
    _check(pkg, np.tile(logits, (copies, 1, 1)), np.tile(labels, (copies, 1)), np.full(B * copies, L, dtype=np.int32),
           np.full(B * copies, T, dtype=np.int32), blank, tol, only=[*range(B)] + [B * copies - 1])


@pytest.mark.parametrize("copies", [1, 130])
@pytest.mark.parametrize("n1,n2,n3,low", [(160, 180, 180, -8.0), (60, 70, 70, -15.0), (40, 45, 45, -26.0), (32, 40, 40, -30.0), (20, 24, 24, -41.0)])
def test_token_spoken_twice_labelled_once(pkg, n1, n2, n3, low, copies):  # noqa: F811
    """The path that counts waits in the first blank while the token, the state beside it, is likely."""
    print(f"ctc_loss twice {n1} {n2} {n3} {low} x {copies}", flush=True)
    logits = np.full((1, n1 + n2 + n3, 3), np.float32(low))
    logits[:, :, 0] = 0.0
    logits[:, n1:n1 + n2, 0], logits[:, n1:n1 + n2, 2] = low, 0.0
    _far(pkg, logits, np.zeros((1, 1), dtype=np.int32), copies, 2)


@pytest.mark.parametrize("copies", [1, 130])
@pytest.mark.parametrize("T,first,run,low", [(100, 1, 40, -27.0), (100, 1, 40, -38.0), (80, 1, 30, -35.0), (140, 1, 62, -30.0),
                                             (300, 50, 75, -26.0), (300, 64, 70, -25.0), (300, 63, 70, -26.0)])
def test_runs_of_one_token_behind_a_likely_one(pkg, T, first, run, low, copies):  # noqa: F811
    """Equal tokens take two frames each, blank and token: both are improbable, the first label's last token stays likely."""
    print(f"ctc_loss runs T={T} {first} + {run} {low} x {copies}", flush=True)
    labels = np.concatenate([np.arange(first) % 2, np.full(run, 2)])[None].astype(np.int32)
    logits = np.full((1, T, 5), np.float32(low))
    last = labels[0, first - 1]
    for t in range(T):
        logits[0, t, labels[0, t] if t < first else last] = 0.0
    _far(pkg, logits, labels, copies, 4)


@pytest.mark.parametrize("wait,L,extra", [(10, 60, 4), (20, 150, 0), (25, 90, 20), (30, 200, 29), (20, 130, 15)])
def test_only_the_path_ahead_arrives_in_time(pkg, wait, L, extra):  # noqa: F811
    """Likely is: wait in the first blank, then a token a frame.  That comes too late (or nearly so), and what counts has gone ahead
    from the start at 2^-38 a frame, hundreds of tokens' worth below what lies behind it."""
    print(f"ctc_loss ahead {wait} {L} {extra}", flush=True)
    T, C = L + extra, 12
    labels = (np.arange(L, dtype=np.int32) % 11)[None]
    logits = np.full((1, T, C), np.float32(-26.0))
    for t in range(T):
        logits[0, t, C - 1 if t < wait or t - wait >= L else labels[0, t - wait]] = 0.0
    _far(pkg, logits, labels, 1, C - 1)


@pytest.mark.parametrize("seed", range(12))
def test_piecewise_constant(pkg, seed):  # noqa: F811
    rng = np.random.Generator(np.random.PCG64(seed))
    B, T, C = 3, int(rng.integers(64, 400)), int(rng.integers(3, 8))
    L = int(rng.integers(1, min(200, T // 2)))
    low = float(rng.uniform(5, 26))
    print(f"ctc_loss piecewise {seed} T={T} L={L} C={C} low={low}", flush=True)
    logits = np.empty((B, T, C), dtype=np.float32)
    for b in range(B):
        t = 0
        while t < T:
            n = int(rng.integers(16, 81))
            logits[b, t:t + n] = rng.uniform(-low, 0.0, C)
            logits[b, t:t + n, rng.integers(C)] = 0.0
            t += n
    labels = rng.integers(0, C - 1, (B, L)).astype(np.int32)
    _far(pkg, logits, labels, 1, C - 1)


# ---- probabilities of exactly 0: what is lost beside a larger value matters once that one is masked out ------------------------
@pytest.mark.parametrize("copies", [1, 130])
@pytest.mark.parametrize("mask", [17, 31, 32, 40, 54, 63, 64, 90])  # within a step of sixteen frames, at its ends
def test_masked_behind_an_improbable_stretch(pkg, mask, copies):  # noqa: F811
    print(f"ctc_loss masked at {mask} x {copies}", flush=True)
    T, low = mask + 24, -27.0  # log2 p = -39, where doubles are taken
    logits = np.full((1, T, 4), np.float32(low))  # tokens 0 and 1 are the label, 2 is another one, 3 the blank
    logits[0, 0, 0] = 0.0
    logits[0, 1:mask, 1] = 0.0
    logits[0, mask] = [0.0, -np.inf, low, -np.inf]
    logits[0, mask + 1:, 1] = 0.0
    _far(pkg, logits, np.array([[0, 1]], dtype=np.int32), copies, 3)


@pytest.mark.parametrize("seed", range(16))
def test_piecewise_constant_with_masks(pkg, seed):  # noqa: F811
    """Segments with tokens masked out that an alignment of the label does not need there; every sequence stays reachable."""
    rng = np.random.Generator(np.random.PCG64(100 + seed))
    B, T, C = 3, int(rng.integers(64, 400)), int(rng.integers(3, 8))
    L = int(rng.integers(1, min(150, T // 3)))
    low = float(rng.uniform(5, 26))
    print(f"ctc_loss masks {seed} T={T} L={L} C={C} low={low}", flush=True)
    labels = rng.integers(0, C - 1, (B, L)).astype(np.int32)
    logits = np.empty((B, T, C), dtype=np.float32)
    for b in range(B):
        # the alignment that stays: a frame for every token, blanks in between
        needed = np.full(T, C - 1)
        at = np.sort(rng.choice(T // 2, L, replace=False)) * 2
        needed[at] = labels[b]
        t = 0
        while t < T:
            n = int(rng.integers(4, 60))
            logits[b, t:t + n] = rng.uniform(-low, 0.0, C)
            logits[b, t:t + n, rng.integers(C)] = 0.0
            masked = rng.random(C) < 0.3
            for u in range(t, min(T, t + n)):
                for c in np.flatnonzero(masked):
                    if c != needed[u]:
                        logits[b, u, c] = -np.inf
            t += n
    _far(pkg, logits, labels, 1, C - 1)


@pytest.mark.parametrize("B,T,L", [(128, 90, 30), (129, 90, 30), (200, 120, 40), (256, 90, 30), (257, 90, 30), (43, 200, 130), (80, 200, 130)])
def test_loss_alone_has_the_same_bits(pkg, B, T, L):  # noqa: F811
    """One direction or two, on both sides of the line between the forms (256 blocks of both directions)."""
    print(f"ctc_loss alone B={B} T={T} L={L}", flush=True)
    rng = np.random.Generator(np.random.PCG64(B))
    C = 50
    args = (dev_f32(rng.standard_normal((B, T, C), dtype=np.float32) * np.float32(2)), dev_i32(rng.integers(0, C - 1, (B, L))),
            dev_i32(rng.integers(L // 2, L + 1, B)), dev_i32(rng.integers(3 * T // 4, T + 1, B)), C - 1)
    ctx = pkg.Context(max_batch=1, max_slots=1, max_topk=1, max_vocab_rows=8, max_nodes=1, max_heads=1, max_head_dim=8)
    assert torch.equal(pkg.ctc_loss(ctx, *args)["loss"], pkg.ctc_loss(ctx, *args, want_grad=False)["loss"])
    ctx.close()
