"""The tile loop with fewer steps than one trip of its pipelined part (hidden sizes below 512): the loop has to end
with every wavefront done reading LDS, because the epilogues put the logit block there."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pkg():
    import paper_2412_00061_amd as pkg
    return pkg


def _operands(seed, cols, D, V):
    g = torch.Generator(device="cuda").manual_seed(seed)
    h = torch.randn((cols, D), generator=g, device="cuda").to(torch.bfloat16)
    w = (torch.randn((V, D), generator=g, device="cuda") * 0.05).to(torch.bfloat16)
    return h, w, (h.double() @ w.double().t()).cpu().numpy()


# float32 sums of D exact products: the error of a sum in any order is below D * 2^-24 of the sum of magnitudes,
# far below 1e-5 of the largest logit at these sizes
@pytest.mark.parametrize("D", [128, 256, 384, 512, 640])
@pytest.mark.parametrize("B,N", [(1, 16), (1, 128), (2, 100)])
def test_verify_head_short_hidden(pkg, D, B, N):
    V = 1300
    h, w, z_ref = _operands(D + N, B * N, D, V)
    ctx = pkg.Context(max_batch=B, max_slots=8, max_topk=4, max_vocab_rows=V, max_nodes=N, max_heads=1, max_head_dim=8)
    n_nodes = torch.full((B,), N, dtype=torch.int32, device="cuda")
    for _ in range(4):
        res = pkg.verify_head_argmax(ctx, h.view(B, N, D), w, n_nodes, want_logits=True)
        z = res["logits"].cpu().numpy().reshape(B * N, V)
        assert np.max(np.abs(z - z_ref)) <= 1e-5 * np.abs(z_ref).max()
        assert np.array_equal(res["target_argmax"].cpu().numpy().reshape(-1), z.argmax(1))
    ctx.close()


@pytest.mark.parametrize("D", [128, 256, 384])
def test_draft_head_short_hidden(pkg, D):
    B, T, Vp1, k = 8, 8, 1301, 4
    h, w, z_ref = _operands(D, B * T, D, Vp1)
    ctx = pkg.Context(max_batch=B, max_slots=T, max_topk=k, max_vocab_rows=Vp1, max_nodes=8, max_heads=1, max_head_dim=8)
    for _ in range(4):
        res = pkg.ctc_draft_topk(ctx, h.view(B, T, D), w, None, k, want_logits=True)
        z = res["logits"].cpu().numpy().reshape(B * T, Vp1)
        assert np.max(np.abs(z - z_ref)) <= 1e-5 * np.abs(z_ref).max()
        top = res["topk_id"].cpu().numpy().reshape(B * T, k)
        assert np.array_equal(top, np.argsort(-z, axis=1, kind="stable")[:, :k])
    ctx.close()
