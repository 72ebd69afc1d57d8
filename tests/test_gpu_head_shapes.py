"""The tile loop of the two heads over sizes where it can go wrong: hidden sizes around its steps and the 16-byte
chunks (rows that start at any element), column counts around the tile widths, a last row block of one row."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

HIDDEN = [1, 7, 8, 60, 64, 65, 100, 127, 129, 264, 500, 513, 1000, 1031]
COLUMNS = [1, 16, 17, 32, 33, 64, 65, 128, 129, 300]


@pytest.fixture(scope="module")
def pkg():
    import paper_2412_00061_amd as pkg
    return pkg


def _operands(seed, cols, D, V, dtype):
    g = torch.Generator(device="cuda").manual_seed(seed)
    h = torch.randn((cols, D), generator=g, device="cuda").to(dtype)
    w = (torch.randn((V, D), generator=g, device="cuda") * 0.05).to(dtype)
    z = h.double() @ w.double().t()
    # a float32 sum of D products in any order, each rounded: at most D + 1 roundings of the sum of magnitudes
    bound = (D + 1) * 2.0 ** -24 * (h.double().abs() @ w.double().abs().t())
    return h, w, z.cpu().numpy(), bound.cpu().numpy()


def _check(z, z_ref, bound):
    assert np.all(np.abs(z - z_ref) <= bound + 1e-30)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("i", range(len(HIDDEN)))
def test_verify_head_any_hidden(pkg, dtype, i):
    D = HIDDEN[i]
    for j, V in ((i, 385), (i + 3, 130), (i + 6, 1)):
        cols = COLUMNS[j % len(COLUMNS)]
        B, N = (3, 100) if cols == 300 else (3, 43) if cols == 129 else (1, cols)
        print(f"verify head {dtype} D={D} V={V} B={B} N={N}", flush=True)
        h, w, z_ref, bound = _operands(100 * i + j, B * N, D, V, dtype)
        ctx = pkg.Context(max_batch=B, max_slots=1, max_topk=1, max_vocab_rows=V, max_nodes=N, max_heads=1, max_head_dim=8)
        n_nodes = torch.full((B,), N, dtype=torch.int32, device="cuda")
        n_nodes[0] = max(1, N - 1)
        res = pkg.verify_head_argmax(ctx, h.view(B, N, D), w, n_nodes, want_logits=True)
        z = res["logits"].cpu().numpy().reshape(B * N, V)
        _check(z, z_ref, bound)
        want = z.argmax(1).reshape(B, N)
        want[0, int(n_nodes[0]):] = -1
        assert np.array_equal(res["target_argmax"].cpu().numpy(), want)
        ctx.close()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("i", range(len(HIDDEN)))
def test_draft_head_any_hidden(pkg, dtype, i):
    D = HIDDEN[i]
    for j, (B, T) in enumerate([(1, 1), (2, 8), (3, 6), (4, 8), (5, 7), (8, 8)]):
        k = 1 + (i + j) % 5
        Vp1 = (130, 385, 257)[(i + j) % 3]
        print(f"draft head {dtype} D={D} Vp1={Vp1} B={B} T={T} k={k}", flush=True)
        h, w, z_ref, bound = _operands(100 * i + j, B * T, D, Vp1, dtype)
        bias = torch.linspace(-1, 1, Vp1, device="cuda")
        ctx = pkg.Context(max_batch=B, max_slots=T, max_topk=k, max_vocab_rows=Vp1, max_nodes=8, max_heads=1, max_head_dim=8)
        res = pkg.ctc_draft_topk(ctx, h.view(B, T, D), w, bias, k, want_logits=True)
        z = res["logits"].cpu().numpy().reshape(B * T, Vp1)
        z_ref = z_ref + bias.double().cpu().numpy()
        _check(z, z_ref, bound + 2.0 ** -23 * (1 + np.abs(z_ref)))
        top = res["topk_id"].cpu().numpy().reshape(B * T, k)
        assert np.array_equal(top, np.argsort(-z, axis=1, kind="stable")[:, :k])
        lse = np.log(np.exp(z.astype(np.float64)).sum(1))
        assert np.max(np.abs(res["lse"].cpu().numpy().reshape(-1) - lse)) <= 2e-5
        ctx.close()


# Vocabularies that do not fill the chip, long hidden dimensions: cut into ranges of the hidden dimension, a column finished
# by one workgroup that holds 1, 2, 4 or 8 groups of rows per thread (2048 rows each).  Every 50th row repeats row 3, so
# the best keys tie across row blocks; a column that has no node; without logits the tokens are the same.
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("B,N,D,V", [(1, 128, 64, 100), (1, 16, 4096, 1500), (3, 43, 2049, 2049), (1, 33, 1031, 4100),
                                     (8, 64, 1000, 4096), (1, 70, 2304, 9000), (2, 64, 5000, 128)])
def test_verify_head_few_rows_long_hidden(pkg, dtype, B, N, D, V):
    print(f"verify head few rows {dtype} D={D} V={V} B={B} N={N}", flush=True)
    h, w, _, _ = _operands(D + V, B * N, D, V, dtype)
    w[3::50] = w[3].clone()
    z_ref = (h.double() @ w.double().t()).cpu().numpy()
    bound = ((D + 1) * 2.0 ** -24 * (h.double().abs() @ w.double().abs().t())).cpu().numpy()
    ctx = pkg.Context(max_batch=B, max_slots=1, max_topk=1, max_vocab_rows=V, max_nodes=N, max_heads=1, max_head_dim=8)
    n_nodes = torch.full((B,), N, dtype=torch.int32, device="cuda")
    n_nodes[B - 1] = N - 1
    res = pkg.verify_head_argmax(ctx, h.view(B, N, D), w, n_nodes, want_logits=True)
    z = res["logits"].cpu().numpy().reshape(B * N, V)
    _check(z, z_ref, bound)
    assert np.array_equal(z[:, 3], z[:, 53])
    want = z.argmax(1).reshape(B, N)
    want[B - 1, N - 1:] = -1
    assert np.array_equal(res["target_argmax"].cpu().numpy(), want)
    assert torch.equal(pkg.verify_head_argmax(ctx, h.view(B, N, D), w, n_nodes)["target_argmax"], res["target_argmax"])
    ctx.close()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("B,T,D,Vp1,k", [(1, 1, 4096, 259, 1), (8, 8, 2048, 1054, 8), (5, 7, 1136, 2048, 6), (3, 6, 768, 2049, 3),
                                         (1, 3, 4608, 129, 2), (7, 1, 4456, 5000, 5), (4, 8, 3000, 8193, 4), (1, 8, 64, 8, 8)])
def test_draft_head_few_rows_long_hidden(pkg, dtype, B, T, D, Vp1, k):
    print(f"draft head few rows {dtype} D={D} Vp1={Vp1} B={B} T={T} k={k}", flush=True)
    h, w, _, _ = _operands(D + Vp1, B * T, D, Vp1, dtype)
    w[3::50] = w[3].clone()
    h[0] = 4 * w[3]  # ties of the largest
    z_ref = (h.double() @ w.double().t()).cpu().numpy()
    bound = ((D + 1) * 2.0 ** -24 * (h.double().abs() @ w.double().abs().t())).cpu().numpy()
    ctx = pkg.Context(max_batch=B, max_slots=T, max_topk=k, max_vocab_rows=Vp1, max_nodes=8, max_heads=1, max_head_dim=8)
    res = pkg.ctc_draft_topk(ctx, h.view(B, T, D), w, None, k, want_logits=True)
    z = res["logits"].cpu().numpy().reshape(B * T, Vp1)
    _check(z, z_ref, bound)
    top = res["topk_id"].cpu().numpy().reshape(B * T, k)
    assert np.array_equal(top, np.argsort(-z, axis=1, kind="stable")[:, :k])
    lse = np.log(np.exp(z.astype(np.float64) - z.max(1, keepdims=True)).sum(1)) + z.max(1)
    # float32 sums of Vp1 terms, and an ulp or two of the largest logit
    tol = 2e-5 + 4 * 2.0 ** -24 * np.abs(z).max(1)
    assert np.all(np.abs(res["lse"].cpu().numpy().reshape(-1) - lse) <= tol)
    logp = np.take_along_axis(z, top, 1) - lse[:, None]
    assert np.all(np.abs(res["topk_logp"].cpu().numpy().reshape(B * T, k) - logp) <= tol[:, None] + 2.0 ** -23 * np.abs(logp))
    ctx.close()


# The heads' own kernels at sizes that the ranges do not take (more than 16384 rows, or hidden dimensions too short for them;
# test_launch_plans.py asks the rule).  Draft head: the tile loop with the epilogue of a lane per column (more than 16
# columns), and the streaming kernel with two to four column tiles (bf16, D a multiple of 512).
DRAFT_OWN_KERNEL = [(5, 8, 256, 16500, "bf16", ("tile", 64, 0)), (8, 8, 520, 16513, "bf16", ("tile", 64, 0)),
                    (3, 8, 261, 16513, "bf16", ("tile", 32, 0)), (5, 8, 256, 16500, "f32", ("tile", 64, 0)),
                    (3, 8, 261, 16513, "f32", ("tile", 32, 0)), (8, 8, 512, 16500, "f32", ("tile", 64, 0)),
                    (3, 7, 512, 17000, "bf16", ("stream", 2, 2)), (3, 7, 1024, 17000, "bf16", ("stream", 2, 4)),
                    (5, 8, 512, 17000, "bf16", ("stream", 3, 2)), (8, 8, 512, 16500, "bf16", ("stream", 4, 2))]
TYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


@pytest.mark.parametrize("B,T,D,Vp1,dtype,way", DRAFT_OWN_KERNEL)
def test_draft_head_own_kernels_every_k(pkg, B, T, D, Vp1, dtype, way):
    h, w, _, _ = _operands(D + Vp1, B * T, D, Vp1, TYPES[dtype])
    # equal rows in one 16-row group, in different ones and in different row blocks: equal logits, ids ascending among them
    equal, second = [3, 5, 19, 131, 900, 16449], [17, 1040]
    w[equal] = w[3].clone()
    w[second] = w[17].clone()
    bias = torch.linspace(-1, 1, Vp1, device="cuda")
    bias[equal], bias[second] = 400.0, 300.0
    z_ref = ((h.double() @ w.double().t()) + bias.double()).cpu().numpy()
    bound = ((D + 1) * 2.0 ** -24 * (h.double().abs() @ w.double().abs().t())).cpu().numpy()
    ctx = pkg.Context(max_batch=B, max_slots=T, max_topk=8, max_vocab_rows=Vp1, max_nodes=8, max_heads=1, max_head_dim=8)
    for k in range(1, 9):
        print(f"draft head own kernel {dtype} D={D} Vp1={Vp1} B={B} T={T} k={k}", flush=True)
        res = pkg.ctc_draft_topk(ctx, h.view(B, T, D), w, bias, k, want_logits=True)
        z = res["logits"].cpu().numpy().reshape(B * T, Vp1)
        _check(z, z_ref, bound + 2.0 ** -23 * (1 + np.abs(z_ref)))
        top = res["topk_id"].cpu().numpy().reshape(B * T, k)
        assert (top == np.array(equal + second)[:k]).all()
        assert np.array_equal(top, np.argsort(-z, axis=1, kind="stable")[:, :k])
        lse = np.log(np.exp(z.astype(np.float64) - z.max(1, keepdims=True)).sum(1)) + z.max(1)
        tol = 2e-5 + 4 * 2.0 ** -24 * np.abs(z).max(1)
        assert np.all(np.abs(res["lse"].cpu().numpy().reshape(-1) - lse) <= tol)
        logp = np.take_along_axis(z, top, 1) - lse[:, None]
        assert np.all(np.abs(res["topk_logp"].cpu().numpy().reshape(B * T, k) - logp) <= tol[:, None] + 2.0 ** -23 * np.abs(logp))
        none = pkg.ctc_draft_topk(ctx, h.view(B, T, D), w, None, k)
        z0 = (h.double() @ w.double().t()).cpu().numpy()
        got = np.take_along_axis(z0, none["topk_id"].cpu().numpy().reshape(B * T, k).astype(np.int64), 1)
        want = -np.sort(-z0, axis=1)[:, :k]
        assert np.all(np.abs(got - want) <= 2 * bound.max(1)[:, None])
    ctx.close()


# Base head: its own kernels with up to 128 columns (128-row tiles) and with more (256-row tiles), several steps and row
# blocks, rows at any alignment; and 128-column tiles of the ranges.
BASE_WIDE = [(1, 16, 256, 17000, "bf16", ("tile", 16, 128)), (1, 30, 512, 17000, "f32", ("tile", 32, 128)), (1, 50, 261, 16999, "bf16", ("tile", 64, 128)),
             (1, 100, 256, 17000, "f32", ("tile", 128, 128)), (1, 100, 261, 16999, "f32", ("tile", 128, 128)),
             (3, 100, 256, 17000, "f32", ("tile", 128, 256)), (4, 50, 1031, 16999, "f32", ("tile", 128, 256)),
             (1, 100, 256, 17000, "bf16", ("tile", 128, 128)), (1, 100, 261, 16999, "bf16", ("tile", 128, 128)),
             (3, 100, 256, 17000, "bf16", ("tile", 128, 256)), (4, 50, 1031, 16999, "bf16", ("tile", 128, 256)),
             (8, 64, 1024, 5000, "f32", ("ranges", 128, 1)), (8, 64, 1031, 5000, "f32", ("ranges", 128, 1)),
             (3, 100, 1031, 2500, "bf16", ("ranges", 128, 2)), (8, 64, 2049, 3000, "bf16", ("ranges", 128, 2))]


@pytest.mark.parametrize("B,N,D,V,dtype,way", BASE_WIDE)
def test_verify_head_many_columns(pkg, B, N, D, V, dtype, way):
    print(f"verify head {way} {dtype} D={D} V={V} B={B} N={N}", flush=True)
    h, w, z_ref, bound = _operands(D + V, B * N, D, V, TYPES[dtype])
    ctx = pkg.Context(max_batch=B, max_slots=1, max_topk=1, max_vocab_rows=V, max_nodes=N, max_heads=1, max_head_dim=8)
    n_nodes = torch.full((B,), N, dtype=torch.int32, device="cuda")
    n_nodes[0] = N - 1
    res = pkg.verify_head_argmax(ctx, h.view(B, N, D), w, n_nodes, want_logits=True)
    z = res["logits"].cpu().numpy().reshape(B * N, V)
    _check(z, z_ref, bound)
    want = z.argmax(1).reshape(B, N)
    want[0, N - 1] = -1
    assert np.array_equal(res["target_argmax"].cpu().numpy(), want)
    assert torch.equal(pkg.verify_head_argmax(ctx, h.view(B, N, D), w, n_nodes)["target_argmax"], res["target_argmax"])
    # equal rows of the largest logit in one row block, in the next and in the last: the smallest id
    h, w = h.abs(), w.clone()
    w[[9, 7, 300, V - 1]] = 0.5
    want[:] = 7
    want[0, N - 1] = -1
    assert np.array_equal(pkg.verify_head_argmax(ctx, h.view(B, N, D), w, n_nodes)["target_argmax"].cpu().numpy(), want)
    ctx.close()


def test_small_contexts_keep_small_scratch(pkg):
    """A context keeps room for the heads' partial sums by its limits, and the heads take the same way in it as in a large one."""
    small = dict(max_batch=1, max_slots=1, max_topk=1, max_vocab_rows=8, max_nodes=8, max_heads=1, max_head_dim=8)
    sizes = []
    for more in ({}, dict(max_vocab_rows=2000, max_slots=8, max_nodes=64)):
        ctx = pkg.Context(**{**small, **more})
        sizes.append(ctx.workspace_bytes())
        ctx.close()
    # the attention's partials and the collapse's tables are 1.3 and 1.6 MB of the first
    assert sizes[0] < 4 << 20 and sizes[1] - sizes[0] < 12 << 20
    large = pkg.Context(max_batch=8, max_slots=8, max_topk=8, max_vocab_rows=40000, max_nodes=64, max_heads=1, max_head_dim=8)
    for B, T, N, D, V, dtype in [(1, 8, 16, 4096, 1500, "bf16"), (2, 8, 64, 1031, 700, "f32"), (1, 1, 1, 2048, 130, "bf16")]:
        print(f"exact context B={B} T={T} N={N} D={D} V={V} {dtype}", flush=True)
        h, w, _, _ = _operands(V, B * N, D, V, TYPES[dtype])
        hd = h.repeat(8, 1)[:B * T].view(B, T, D).contiguous()
        n_nodes = torch.full((B,), N, dtype=torch.int32, device="cuda")
        exact = pkg.Context(max_batch=B, max_slots=T, max_topk=4, max_vocab_rows=V, max_nodes=N, max_heads=1, max_head_dim=8)
        for call in (lambda c: pkg.verify_head_argmax(c, h.view(B, N, D), w, n_nodes, want_logits=True),
                     lambda c: pkg.ctc_draft_topk(c, hd, w, None, 4, want_logits=True)):
            a, b = call(exact), call(large)
            assert all(torch.equal(a[n], b[n]) for n in a)
        exact.close()
    large.close()
