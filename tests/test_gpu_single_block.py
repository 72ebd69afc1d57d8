"""Heads whose vocabulary is a single row block finish themselves in one launch: every tile width, short and long rows, as many
rows as k, columns without a node, ties, and a deferred merge that leaves nothing owed."""
import numpy as np
import pytest
import torch

from test_gpu_head_shapes import TYPES, _check, _operands, pkg  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V", [1, 5, 100, 127, 128, 129])
def test_base_head(pkg, dtype, V):  # noqa: F811
    for B, N, D in ((1, 1, 64), (1, 16, 128), (1, 17, 40), (3, 43, 64), (8, 64, 65), (2, 100, 512)):
        print(f"single block base head {dtype} D={D} V={V} B={B} N={N}", flush=True)
        h, w, z_ref, bound = _operands(V + D, B * N, D, V, TYPES[dtype])
        ctx = pkg.Context(max_batch=B, max_slots=1, max_topk=1, max_vocab_rows=V, max_nodes=N, max_heads=1, max_head_dim=8)
        n_nodes = torch.full((B,), N, dtype=torch.int32, device="cuda")
        n_nodes[B - 1] = max(1, N - 2)
        res = pkg.verify_head_argmax(ctx, h.view(B, N, D), w, n_nodes, want_logits=True)
        z = res["logits"].cpu().numpy().reshape(B * N, V)
        _check(z, z_ref, bound)
        want = z.argmax(1).reshape(B, N)
        want[B - 1, int(n_nodes[B - 1]):] = -1
        assert np.array_equal(res["target_argmax"].cpu().numpy(), want)
        w[[0, V - 1]] = w[V // 2].clone()  # ties
        res = pkg.verify_head_argmax(ctx, h.view(B, N, D), w, n_nodes, want_logits=True)
        want = res["logits"].cpu().numpy().reshape(B * N, V).argmax(1).reshape(B, N)
        want[B - 1, int(n_nodes[B - 1]):] = -1
        assert np.array_equal(res["target_argmax"].cpu().numpy(), want)
        ctx.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("Vp1", [5, 101, 127, 128, 129])
def test_draft_head(pkg, dtype, Vp1):  # noqa: F811
    for B, T, D, k in ((1, 1, 64, 1), (1, 4, 64, 2), (2, 8, 256, 5), (3, 8, 64, 4), (8, 8, 512, 5), (1, 8, 1024, 3)):
        print(f"single block draft head {dtype} D={D} Vp1={Vp1} B={B} T={T} k={k}", flush=True)
        h, w, _, _ = _operands(Vp1 + D, B * T, D, Vp1, TYPES[dtype])
        w[[0, Vp1 - 1]] = w[Vp1 // 2].clone()
        bias = torch.zeros(Vp1, device="cuda")
        ctx = pkg.Context(max_batch=B, max_slots=T, max_topk=k, max_vocab_rows=Vp1, max_nodes=8, max_heads=1, max_head_dim=8)
        results = []
        for defer in (False, True):
            ctx.defer_topk_merge(defer)
            res = pkg.ctc_draft_topk(ctx, h.view(B, T, D), w, bias, k, want_logits=True)
            ctx.flush()
            results.append({n: t.cpu().numpy().reshape(B * T, -1) for n, t in res.items()})
        a, b = results
        assert all(np.array_equal(a[n], b[n]) for n in a)
        z = a["logits"]
        z_ref = (h.double() @ w.double().t()).cpu().numpy()
        _check(z, z_ref, (D + 1) * 2.0 ** -24 * (h.double().abs() @ w.double().abs().t()).cpu().numpy() + 2.0 ** -23 * (1 + np.abs(z_ref)))
        top = np.argsort(-z, axis=1, kind="stable")[:, :k]
        assert np.array_equal(a["topk_id"], top)
        lse = np.log(np.exp(z.astype(np.float64) - z.max(1, keepdims=True)).sum(1)) + z.max(1)
        tol = 2e-5 + 4 * 2.0 ** -24 * np.abs(z).max(1)
        assert np.all(np.abs(a["lse"][:, 0] - lse) <= tol)
        logp = np.take_along_axis(z, top, 1) - lse[:, None]
        assert np.all(np.abs(a["topk_logp"] - logp) <= tol[:, None] + 2.0 ** -23 * np.abs(logp))
        ctx.close()
