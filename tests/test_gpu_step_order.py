"""Rows a multiple of 4096 bytes apart are walked in steps 2048 bytes apart: every kernel of the heads on such rows (two, three and
eight laps, ranges that end within a lap), logits against float64 and equal weight rows in different row blocks bit for bit."""
import numpy as np
import pytest
import torch

from test_gpu_head_shapes import TYPES, _check, _operands, pkg  # noqa: F401

pytestmark = pytest.mark.gpu

# dtype, hidden size: rows of 4096, 8192, 12288 and 16384 bytes
ROWS = [("bf16", 2048), ("bf16", 4096), ("bf16", 6144), ("f32", 1024), ("f32", 3072)]


@pytest.mark.parametrize("dtype,D", ROWS)
@pytest.mark.parametrize("cols", [5, 30, 60, 100, 200])
@pytest.mark.parametrize("V", [16400, 1500])  # the heads' own kernels; ranges of the hidden dimension
def test_base_head_rows_of_4096_bytes(pkg, dtype, D, cols, V):  # noqa: F811
    print(f"base head {dtype} D={D} V={V} cols={cols}", flush=True)
    B, N = (2, cols // 2) if cols > 128 else (1, cols)
    h, w, _, _ = _operands(D + cols, cols, D, V, TYPES[dtype])
    w[[9, 700, V - 1]] = w[9].clone()
    z_ref = (h.double() @ w.double().t()).cpu().numpy()
    bound = ((D + 1) * 2.0 ** -24 * (h.double().abs() @ w.double().abs().t())).cpu().numpy()
    ctx = pkg.Context(max_batch=B, max_slots=1, max_topk=1, max_vocab_rows=V, max_nodes=N, max_heads=1, max_head_dim=8)
    n_nodes = torch.full((B,), N, dtype=torch.int32, device="cuda")
    res = pkg.verify_head_argmax(ctx, h.view(B, N, D), w, n_nodes, want_logits=True)
    z = res["logits"].cpu().numpy().reshape(cols, V)
    _check(z, z_ref, bound)
    assert np.array_equal(z[:, 9], z[:, 700]) and np.array_equal(z[:, 9], z[:, V - 1])
    assert np.array_equal(res["target_argmax"].cpu().numpy().reshape(-1), z.argmax(1))
    ctx.close()


@pytest.mark.parametrize("dtype,D", ROWS + [("bf16", 8192)])
@pytest.mark.parametrize("B,T", [(1, 8), (2, 8), (3, 8), (8, 8)])
def test_draft_head_rows_of_4096_bytes(pkg, dtype, D, B, T):  # noqa: F811
    Vp1, k = 16400, 4
    print(f"draft head {dtype} D={D} Vp1={Vp1} B={B} T={T}", flush=True)
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
