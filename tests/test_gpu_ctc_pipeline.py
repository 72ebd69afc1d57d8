"""ctc_loss with frames enough for the pipelined recursions: labels around the blocks of 64 pairs of states, frame counts
around the 16 frames of a step and the rule's limit, probabilities of zero, and tokens masked out by large finite
numbers, for which the recursion runs in the log domain."""
import math

import numpy as np
import pytest
import torch

import oracle
from gpu_harness import rel_err_rms_floor
from workloads.device import dev_f32, dev_i32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pkg():
    import paper_2412_00061_amd as m
    return m


def _check(pkg, logits, labels, label_len, frame_len, blank, grad_tol=1e-4, only=None, reference=oracle.ctc_loss_and_grad):
    B, T, C = logits.shape
    ctx = pkg.Context(max_batch=1, max_slots=1, max_topk=1, max_vocab_rows=8, max_nodes=1, max_heads=1, max_head_dim=8)
    args = (dev_f32(logits), dev_i32(labels), dev_i32(label_len), dev_i32(frame_len), blank)
    res = pkg.ctc_loss(ctx, *args)
    again = pkg.ctc_loss(ctx, *args)
    alone = pkg.ctc_loss(ctx, *args, want_grad=False)
    loss, grad = res["loss"].cpu().numpy(), res["grad"].cpu().numpy()
    assert torch.equal(res["loss"], again["loss"]) and torch.equal(res["grad"].view(torch.int32), again["grad"].view(torch.int32))
    assert torch.equal(res["loss"], alone["loss"])
    for b in range(B) if only is None else only:
        Tb, L = int(frame_len[b]), int(label_len[b])
        if Tb == 0:  # no frame: the empty label is certain
            assert loss[b] == (0.0 if L == 0 else math.inf) and not grad[b].any()
            continue
        ref_loss, ref_grad = reference(logits[b, :Tb], tuple(int(v) for v in labels[b, :L]), blank)
        assert not grad[b, Tb:].any()
        if math.isinf(ref_loss):
            assert math.isinf(loss[b]) and not grad[b].any()
            continue
        # bars of the loss's other tests: a few ulps of the loss, 1e-4 of max(|entry|, rms) of the gradient
        assert abs(loss[b] - ref_loss) <= 2e-6 * max(1.0, abs(ref_loss)), (b, loss[b], ref_loss)
        if ref_loss > 1e6:  # a masked-out token is needed: float32 log-probabilities of that size are whole numbers
            continue
        assert rel_err_rms_floor(grad[b, :Tb], ref_grad) <= grad_tol, (b, rel_err_rms_floor(grad[b, :Tb], ref_grad))
    ctx.close()


@pytest.mark.parametrize("T", [63, 64, 65, 80, 81, 300])
@pytest.mark.parametrize("L", [0, 1, 62, 63, 64, 65, 127, 128, 130])
def test_blocks_and_steps(pkg, T, L):
    rng = np.random.Generator(np.random.PCG64(1000 * T + L))
    B, C, Lmax = 3, 23, max(L, 1)
    print(f"ctc_loss T={T} L={L}", flush=True)
    logits = rng.standard_normal((B, T, C), dtype=np.float32) * np.float32(1.5)
    labels = rng.integers(0, C - 1, size=(B, Lmax)).astype(np.int32)
    frame_len = np.array([T, max(1, T - 17), 0], dtype=np.int32)
    _check(pkg, logits, labels, np.array([L, L // 2, 0], dtype=np.int32), frame_len, C - 1)


# Sequences without frames at every place of the batch, the first among them (its rows return early, and the call's
# bookkeeping must not hang on them), in a workspace that other bytes or another shape's call have been in before.
@pytest.mark.parametrize("frames", [(0, 90, 73), (0, 0, 0), (90, 0, 73), (0, 0, 90)])
@pytest.mark.parametrize("T,Lmax", [(90, 20), (90, 130), (20, 7)])
def test_empty_sequences(pkg, frames, T, Lmax):
    rng = np.random.Generator(np.random.PCG64(11 * T + Lmax + frames[0]))
    B, C = 3, 23
    frame_len = np.minimum(np.array(frames, dtype=np.int32), T)
    logits = rng.standard_normal((B, T, C), dtype=np.float32) * np.float32(1.5)
    labels = rng.integers(0, C - 1, size=(B, Lmax)).astype(np.int32)
    label_len = np.array([min(5, Lmax), 0, min(20, Lmax)], dtype=np.int32)
    ctx = pkg.Context(max_batch=1, max_slots=1, max_topk=1, max_vocab_rows=8, max_nodes=1, max_heads=1, max_head_dim=8)
    other = (dev_f32(rng.standard_normal((2, 70, C), dtype=np.float32)), dev_i32(labels[:2, :7]), dev_i32(label_len[:2]),
             dev_i32(np.array([70, 64])), C - 1)
    args = (dev_f32(logits), dev_i32(labels), dev_i32(label_len), dev_i32(frame_len), C - 1)
    need = max(pkg.ctc_loss_workspace_bytes(B, T, Lmax), pkg.ctc_loss_workspace_bytes(2, 70, 7))
    for fill in (0xFF, 0x00, 0x01, None):
        print(f"ctc_loss T={T} Lmax={Lmax} frames={frame_len.tolist()} fill={fill}", flush=True)
        ws = torch.full((need,), fill or 0, dtype=torch.uint8, device="cuda")
        if fill is None:
            pkg.ctc_loss(ctx, *other, workspace=ws)
        out = {"loss": torch.full((B,), -7.0, device="cuda"), "grad": torch.full((B, T, C), -7.0, device="cuda")}
        for want_grad in (True, False):
            if fill is not None:
                ws.fill_(fill)
            res = pkg.ctc_loss(ctx, *args, want_grad=want_grad, workspace=ws, out=out)
            loss = res["loss"].cpu().numpy()
            for b in range(B):
                Tb, L = int(frame_len[b]), int(label_len[b])
                if Tb == 0:
                    ref_loss, ref_grad = (0.0 if L == 0 else math.inf), np.zeros((0, C))
                else:
                    ref_loss, ref_grad = oracle.ctc_loss_and_grad(logits[b, :Tb], tuple(int(v) for v in labels[b, :L]), C - 1)
                assert loss[b] == ref_loss or abs(loss[b] - ref_loss) <= 2e-6 * max(1.0, abs(ref_loss)), (b, loss[b], ref_loss)
                if want_grad:
                    grad = res["grad"][b].cpu().numpy()
                    assert not grad[Tb:].any()
                    assert Tb == 0 or rel_err_rms_floor(grad[:Tb], ref_grad) <= 1e-4
            out["loss"].fill_(-7.0)
    ctx.close()


# Logits that are no numbers (a diverged run): the loss of such a sequence is not a number - not +inf, which stands for a
# label that cannot be reached - and its gradient zero; the other sequences of the batch do not notice.  One wavefront per
# sequence (few frames; many short labels), one block of states and several, with and without a token masked by a
# large finite number (the log-domain recursion), and a label that could not be reached anyway (no repeats fit).
@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("B,T,L,masked", [(3, 20, 6, False), (800, 70, 6, False), (3, 90, 20, False), (3, 300, 130, False),
                                          (3, 90, 20, True), (3, 300, 130, True), (3, 70, 69, False),
                                          (3, 12, 70, False), (3, 20, 70, False)])
def test_not_a_number(pkg, bad, B, T, L, masked):
    rng = np.random.Generator(np.random.PCG64(17 * T + L))
    C = 23
    print(f"ctc_loss B={B} T={T} L={L} masked={masked} bad={bad}", flush=True)
    logits = rng.standard_normal((B, T, C), dtype=np.float32)
    labels = rng.integers(0, C - 1, size=(B, L)).astype(np.int32)
    if masked:
        logits[:2, ::4, labels[0, 2]] = -1e9
    clean = logits.copy()
    logits[0, T // 2, 5] = bad
    logits[1, T - 1, :] = bad  # behind the sequence's frames
    ctx = pkg.Context(max_batch=1, max_slots=1, max_topk=1, max_vocab_rows=8, max_nodes=1, max_heads=1, max_head_dim=8)
    frame_len = np.full(B, T, dtype=np.int32)
    frame_len[1] = T - 1
    rest = (dev_i32(labels), dev_i32(np.full(B, L, dtype=np.int32)), dev_i32(frame_len), C - 1)
    got, want = pkg.ctc_loss(ctx, dev_f32(logits), *rest), pkg.ctc_loss(ctx, dev_f32(clean), *rest)
    alone = pkg.ctc_loss(ctx, dev_f32(logits), *rest, want_grad=False)
    assert torch.isnan(got["loss"][0]) and torch.isnan(alone["loss"][0]) and not got["grad"][0].any()
    assert torch.equal(got["loss"][1:], want["loss"][1:]) and torch.equal(alone["loss"][1:], want["loss"][1:])
    assert torch.equal(got["grad"][1:], want["grad"][1:])
    assert not torch.isnan(want["loss"]).any()
    ctx.close()


@pytest.mark.parametrize("mask", [-np.inf, -3.0e38, -1e38, -1e9, -1e4])
def test_masked_tokens(pkg, mask):
    # sequence 0: a label's token masked out in half of the frames, where other tokens can take its place; sequence 1: in
    # all frames (unreachable, or a huge loss); sequence 2: nothing of its own masked; sequence 3: the blank masked
    rng = np.random.Generator(np.random.PCG64(5))
    B, T, C, L = 4, 90, 12, 20
    logits = rng.standard_normal((B, T, C), dtype=np.float32)
    labels = np.tile(np.arange(L, dtype=np.int32) % 10, (B, 1))
    logits[0, ::2, 3] = mask
    logits[1, :, 4] = mask
    logits[2, :, 10] = mask
    logits[3, 10:20, 11] = mask
    # a huge loss leaves the float32 log-probabilities themselves a coarse grid: only the loss is compared then; at -1e4
    # they are near 2^14 in base 2, half an ulp is 2^-11, and an occupancy is formed from four such terms: 1.4e-3 of it,
    # five times that of the row's rms where the rms is a fifth of the occupancy
    huge = -np.inf < mask <= -1e9
    n = np.full(B, L, dtype=np.int32)
    f = np.full(B, T, dtype=np.int32)
    if huge:
        keep = [0, 2, 3]
        _check(pkg, logits[keep], labels[keep], n[keep], f[keep], 11)
        ctx = pkg.Context(max_batch=1, max_slots=1, max_topk=1, max_vocab_rows=8, max_nodes=1, max_heads=1, max_head_dim=8)
        res = pkg.ctc_loss(ctx, dev_f32(logits[1:2]), dev_i32(labels[1:2]), dev_i32(n[:1]), dev_i32(f[:1]), 11)
        ref, _ = oracle.ctc_loss_and_grad(logits[1], tuple(int(v) for v in labels[1]), 11)
        got = float(res["loss"][0])
        # (2 log2 e * 3e38 is past the largest float: such a token counts as impossible)
        assert got == math.inf if mask < -2e38 else abs(got - ref) <= 2e-6 * ref
        ctx.close()
    else:
        _check(pkg, logits, labels, n, f, 11, 7e-3 if mask == -1e4 else 1e-4)


def test_peaked_logits_far_from_the_diagonal(pkg):
    # the greedy path says all blanks for most of the sequence, the label is long: the states that matter lie far below
    # the frame's largest alpha or beta.  Exponents within 64 pairs of states spread over 64 x 36: the float32 values held
    # against the block's largest have ulps of 2^-12, half of one in each of alpha and beta, 2^-12 ln 2 = 1.7e-4 of an
    # occupancy, before the occupancies of a frame are divided by their sum
    rng = np.random.Generator(np.random.PCG64(6))
    B, T, C, L = 2, 400, 30, 150
    logits = rng.standard_normal((B, T, C), dtype=np.float32)
    logits[:, :, 29] += 25.0
    logits[1, 200:, 29] -= 50.0
    labels = rng.integers(0, 29, size=(B, L)).astype(np.int32)
    _check(pkg, logits, labels, np.full(B, L, dtype=np.int32), np.full(B, T, dtype=np.int32), 29, 5e-4)


@pytest.mark.parametrize("B,T,Lmax", [(800, 70, 20), (800, 64, 63), (5, 63, 63), (5, 63, 200), (3, 1, 1), (4, 9, 5), (2, 16, 17),
                                      (441, 63, 63), (441, 63, 200), (65, 16, 17), (64, 16, 17), (2, 15, 17), (3, 17, 130)])
def test_wavefront_per_sequence(pkg, B, T, Lmax):
    # few frames (rows in LDS, labels longer than the frames can hold), and many short labels (rows in the workspace);
    # few tokens, so that labels repeat them.  On both sides of the rule's lines: at 16 and 63 frames the pipeline takes up
    # to 64 and 440 sequences
    rng = np.random.Generator(np.random.PCG64(7 * T + Lmax))
    C = 9
    print(f"ctc_loss B={B} T={T} Lmax={Lmax}", flush=True)
    logits = rng.standard_normal((B, T, C), dtype=np.float32) * np.float32(1.5)
    logits[0, : T // 2, 2] = -np.inf
    logits[1, : T // 2, 3] = -1e9
    labels = rng.integers(0, C - 1, size=(B, Lmax)).astype(np.int32)
    frame_len = rng.integers(max(1, T // 2), T + 1, size=B).astype(np.int32)
    label_len = rng.integers(0, np.minimum(Lmax, frame_len) + 1, size=B).astype(np.int32)
    label_len[-1] = Lmax
    keep = [0, 1, B - 1] if B > 10 else range(B)
    _check(pkg, logits, labels, label_len, frame_len, C - 1, only=keep)


@pytest.mark.parametrize("C,T,Lmax", [(2049, 5, 128), (2052, 5, 127), (8193, 6, 511), (8200, 6, 512), (9000, 70, 1100), (40000, 3, 3)])
def test_row_workgroups(pkg, C, T, Lmax):
    # vocabularies and label capacities around the sizes at which a row's workgroup gets more threads
    rng = np.random.Generator(np.random.PCG64(C + Lmax))
    B = 2
    print(f"ctc_loss V+1={C} T={T} Lmax={Lmax}", flush=True)
    logits = rng.standard_normal((B, T, C), dtype=np.float32)
    labels = rng.integers(0, C - 1, size=(B, Lmax)).astype(np.int32)
    _check(pkg, logits, labels, np.array([min(Lmax, T // 2), 1], dtype=np.int32), np.array([T, T - 1], dtype=np.int32), C - 1)


def _torch_reference(logits, label, blank):  # (the oracle takes a minute for 2047 labels)
    x = torch.tensor(logits, dtype=torch.float64, requires_grad=True)
    args = torch.tensor(label)[None], torch.tensor([len(logits)]), torch.tensor([len(label)])
    loss = torch.nn.functional.ctc_loss(torch.log_softmax(x, 1)[:, None], *args, blank=blank, reduction="sum")
    loss.backward()
    return loss.item(), x.grad.numpy()


@pytest.mark.parametrize("L", [1, 63, 64, 255, 256, 511, 512, 1279, 1280, 2047])
def test_log_domain_sizes(pkg, L):
    # a token of the label masked out by a large finite number in every fourth frame, so that the recursion runs in the log
    # domain: one block of states and many, labels that end with a block and in the middle of one, and the largest.
    # The states that matter lie up to 0.2 T bits below a frame's largest (float64 recursions of these inputs: 399 at
    # T = 1938, 616 at 3090); float32 rounds such a value by 0.2 T 2^-24 at most, once per frame, which adds up as a
    # random walk over T frames; ln 2 turns bits into a relative error of the occupancy
    rng = np.random.Generator(np.random.PCG64(31 + L))
    B, T, C = 2, max(70, L + L // 2 + 20), 97
    print(f"ctc_loss T={T} L={L}", flush=True)
    logits = rng.standard_normal((B, T, C), dtype=np.float32)
    labels = rng.integers(0, C - 1, size=(B, L)).astype(np.int32)
    logits[0, ::4, labels[0, L // 2]] = -1e9
    logits[1, 1::4, labels[1, 0]] = -1e9
    _check(pkg, logits, labels, np.array([L, max(1, L - 1)], dtype=np.int32), np.array([T, T - 3], dtype=np.int32), C - 1,
           grad_tol=max(1e-4, 0.2 * T * 2.0**-24 * math.sqrt(T) * math.log(2)), reference=_torch_reference)
