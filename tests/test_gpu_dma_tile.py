"""The tile loop that loads straight into LDS, at the sizes where it can go wrong: fewer steps than its rings have slots and a few
more, rows that end 16 bytes into a step, ragged row and column blocks of every tile shape, 256 x 256 tiles with and without
logits."""
import numpy as np
import pytest
import torch

from test_gpu_head_shapes import TYPES, _check, _operands, pkg  # noqa: F401

pytestmark = pytest.mark.gpu

ROW_BYTES = [272, 512, 640, 784, 1024, 1296, 1552, 2320]  # 2 to 10 steps of 256 bytes (3 to 19 of 128), whole or 16 to 144 bytes over


def _case(pkg, dtype, cols, D, V):  # noqa: F811
    print(f"dma tile {dtype} D={D} V={V} cols={cols}", flush=True)
    B = {200: 2, 520: 8, 732: 6}.get(cols, 1)
    N = cols // B
    h, w, _, _ = _operands(D + cols, cols, D, V, TYPES[dtype])
    same = 700 if V > 700 else V // 2
    w[[9, same, V - 1]] = w[9].clone()
    z_ref = (h.double() @ w.double().t()).cpu().numpy()
    bound = ((D + 1) * 2.0 ** -24 * (h.double().abs() @ w.double().abs().t())).cpu().numpy()
    ctx = pkg.Context(max_batch=B, max_slots=1, max_topk=1, max_vocab_rows=V, max_nodes=N, max_heads=1, max_head_dim=8)
    n_nodes = torch.full((B,), N, dtype=torch.int32, device="cuda")
    n_nodes[0] = max(1, N - 1)
    res = pkg.verify_head_argmax(ctx, h.view(B, N, D), w, n_nodes, want_logits=True)
    z = res["logits"].cpu().numpy().reshape(cols, V)
    _check(z, z_ref, bound)
    assert np.array_equal(z[:, 9], z[:, same]) and np.array_equal(z[:, 9], z[:, V - 1])
    want = z.argmax(1).reshape(B, N)
    want[0, int(n_nodes[0]):] = -1
    assert np.array_equal(res["target_argmax"].cpu().numpy(), want)
    assert torch.equal(pkg.verify_head_argmax(ctx, h.view(B, N, D), w, n_nodes)["target_argmax"], res["target_argmax"])
    ctx.close()


@pytest.mark.parametrize("dtype,elem", [("bf16", 2), ("f32", 4)])
@pytest.mark.parametrize("row", ROW_BYTES)
def test_every_shape(pkg, dtype, elem, row):  # noqa: F811
    for cols in (7, 32, 50, 128, 200):  # (200: two column blocks of 128, 256 rows)
        _case(pkg, dtype, cols, row // elem, 16500)


# 65 row blocks of 256: five column blocks of 128 take two rounds over the compute units, three of 256 one
@pytest.mark.parametrize("dtype,elem", [("bf16", 2), ("f32", 4)])
@pytest.mark.parametrize("row", [272, 640, 1296])
@pytest.mark.parametrize("cols", [520, 732])
def test_tiles_of_256_columns(pkg, dtype, elem, row, cols):  # noqa: F811
    _case(pkg, dtype, cols, row // elem, 16500)


@pytest.mark.parametrize("dtype,elem", [("bf16", 2), ("f32", 4)])
@pytest.mark.parametrize("row", ROW_BYTES)
def test_draft_head_shapes(pkg, dtype, elem, row):  # noqa: F811
    D, Vp1, k = row // elem, 16500, 4
    for B, T in ((1, 5), (3, 7), (5, 8)):
        print(f"dma tile draft head {dtype} D={D} B={B} T={T}", flush=True)
        h, w, _, _ = _operands(D + B, B * T, D, Vp1, TYPES[dtype])
        w[[9, 700, Vp1 - 1]] = w[9].clone()
        z_ref = (h.double() @ w.double().t()).cpu().numpy()
        bound = ((D + 1) * 2.0 ** -24 * (h.double().abs() @ w.double().abs().t())).cpu().numpy()
        ctx = pkg.Context(max_batch=B, max_slots=T, max_topk=k, max_vocab_rows=Vp1, max_nodes=8, max_heads=1, max_head_dim=8)
        res = pkg.ctc_draft_topk(ctx, h.view(B, T, D), w, None, k, want_logits=True)
        z = res["logits"].cpu().numpy().reshape(B * T, Vp1)
        _check(z, z_ref, bound)
        assert np.array_equal(z[:, 9], z[:, 700]) and np.array_equal(z[:, 9], z[:, Vp1 - 1])
        assert np.array_equal(res["topk_id"].cpu().numpy().reshape(B * T, k), np.argsort(-z, axis=1, kind="stable")[:, :k])
        ctx.close()


# Ranges of the hidden dimension of a single step each go through registers, rows on 16-byte boundaries or not (test_launch_plans.py
# asks the rule): columns, hidden size, vocabulary rows
SINGLE_STEPS = [("f32", 20, 256, 975), ("f32", 20, 192, 465), ("f32", 7, 320, 129), ("bf16", 50, 384, 465), ("bf16", 128, 512, 129),
                ("f32", 200, 128, 465)]


@pytest.mark.parametrize("dtype,cols,D,V", SINGLE_STEPS)
def test_ranges_of_a_single_step(pkg, dtype, cols, D, V):  # noqa: F811
    _case(pkg, dtype, cols, D, V)
