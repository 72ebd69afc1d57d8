"""tree_verify_attn with float operands and with head dimensions other than 128: padded head dimensions, tiles and
blocks at their edges, key splits, scores that move the softmax reference, any sign of the scale."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from gpu_harness import dev_i32, dev_i64, rel_err_rms_floor, to_device
from test_gpu_attn_peaked import _trees

pytestmark = pytest.mark.gpu

# (B, H, max_nodes, kv_cap, context lengths): tiles of 32 keys and blocks of 64 rows at their edges, no context at all,
# one key range and up to eight
SHAPES = [(1, 2, 1, 8, [0]), (2, 3, 5, 40, [1, 33]), (1, 4, 16, 64, [31]), (3, 2, 17, 64, [32, 0, 64]),
          (2, 2, 64, 300, [300, 65]), (1, 5, 65, 900, [700]), (2, 12, 100, 900, [300, 900]), (8, 32, 128, 96, [96] * 8)]


@pytest.fixture(scope="module")
def pkg():
    import paper_2412_00061_amd as m
    return m


# Scores are float32 sums of dh products and P has 24 bits: an error of a few 2^-24 of the largest score (about 5 at
# q_scale 1, about 60 at 12) in the exponent, and the float32 sums over the keys behind it
@pytest.mark.parametrize("dtype,dh", [("bf16", d) for d in (8, 16, 40, 64, 72, 96, 104)] +
                         [("f32", d) for d in (8, 16, 40, 64, 80, 96, 120, 128)])
@pytest.mark.parametrize("q_scale,sign,tol", [(1.0, 1.0, 1e-5), (12.0, 1.0, 1e-4), (1.0, -1.0, 1e-5)])
def test_attention_any(pkg, dtype, dh, q_scale, sign, tol):
    for i, (B, H, N, cap, ctx_len) in enumerate(SHAPES):
        if (q_scale > 1 and N < 64) or (sign < 0 and i % 2) or (B == 8 and dh != 64):
            continue
        print(f"attention {dtype} dh={dh} B={B} H={H} N={N} ctx={ctx_len} q_scale={q_scale} sign={sign}", flush=True)
        case = workloads.make_attention_case(i, B, H, N, dh, cap, ctx_len, dtype, q_scale=q_scale)
        trees = _trees(i, B, N, 128, "chain" if N < 8 else "beam")
        n_nodes = np.array([t["n_nodes"] for t in trees], dtype=np.int32)
        q, kt, vt = case.q.copy(), case.k_tree.copy(), case.v_tree.copy()
        for b in range(B):  # rows beyond the tree may hold anything
            q[b, :, n_nodes[b]:] = kt[b, :, n_nodes[b]:] = vt[b, :, n_nodes[b]:] = np.nan
        mask = torch.from_numpy(np.stack([t["anc_mask"] for t in trees]).view(np.int64)).cuda()
        scale = sign / np.sqrt(dh)
        ctx = pkg.Context(max_batch=B, max_slots=1, max_topk=1, max_vocab_rows=8, max_nodes=N, max_heads=H, max_head_dim=dh)
        args = (to_device(q, dtype), to_device(case.k_cache, dtype), to_device(case.v_cache, dtype), dev_i64(case.kv_off),
                dev_i32(case.ctx_len), cap, to_device(kt, dtype), to_device(vt, dtype), dev_i32(n_nodes), mask, scale)
        out = pkg.tree_verify_attn(ctx, *args)
        again = pkg.tree_verify_attn(ctx, *args)
        out, again = out.cpu().numpy(), again.cpu().numpy()
        for b in range(B):
            n = int(n_nodes[b])
            ref = oracle.tree_attention(case.q[b], case.k_cache[b], case.v_cache[b], int(case.ctx_len[b]), case.k_tree[b],
                                        case.v_tree[b], n, trees[b]["mask"], scale)
            assert np.isfinite(out[b, :, :n]).all()
            assert rel_err_rms_floor(out[b, :, :n], ref) <= tol
            assert np.array_equal(out[b, :, :n], again[b, :, :n])
        ctx.close()


# Values that are infinite or not a number: they belong to the rows that see their key, in their own component, and to
# no other - a leaf's value (seen by that node alone) and a cached one (seen by every row, an infinity stays one).
@pytest.mark.parametrize("dtype,dh", [("f32", 64), ("f32", 40), ("f32", 128), ("bf16", 64), ("bf16", 96)])
@pytest.mark.parametrize("B,H,N,cap,ctx_len", [(2, 3, 17, 64, [40, 0]), (2, 3, 100, 900, [900, 300]), (1, 2, 64, 700, [333])])
def test_attention_values_not_finite(pkg, dtype, dh, B, H, N, cap, ctx_len):
    case = workloads.make_attention_case(N, B, H, N, dh, cap, ctx_len, dtype)
    trees = _trees(N, B, N, 128, "beam")
    n_nodes = np.array([t["n_nodes"] for t in trees], dtype=np.int32)
    vt, vc = case.v_tree.copy(), case.v_cache.copy()
    for b in range(B):
        vt[b, :, n_nodes[b] - 1, 3], vt[b, :, n_nodes[b] - 1, 5], vt[b, :, n_nodes[b] - 1, 7] = np.inf, np.nan, -np.inf
    vc[0][:, 2, 1] = np.inf
    print(f"attention not finite {dtype} dh={dh} B={B} H={H} N={N} ctx={ctx_len}", flush=True)
    mask = torch.from_numpy(np.stack([t["anc_mask"] for t in trees]).view(np.int64)).cuda()
    ctx = pkg.Context(max_batch=B, max_slots=1, max_topk=1, max_vocab_rows=8, max_nodes=N, max_heads=H, max_head_dim=dh)
    out = pkg.tree_verify_attn(ctx, to_device(case.q, dtype), to_device(case.k_cache, dtype), to_device(vc, dtype),
                               dev_i64(case.kv_off), dev_i32(case.ctx_len), cap, to_device(case.k_tree, dtype),
                               to_device(vt, dtype), dev_i32(n_nodes), mask, dh ** -0.5).cpu().numpy()
    for b in range(B):
        n = int(n_nodes[b])
        ref = oracle.tree_attention(case.q[b], case.k_cache[b], case.v_cache[b], int(case.ctx_len[b]), case.k_tree[b],
                                    case.v_tree[b], n, trees[b]["mask"], dh ** -0.5)
        got = out[b, :, :n].copy()
        last = got[:, n - 1]
        assert np.isposinf(last[:, 3]).all() and np.isnan(last[:, 5]).all() and np.isneginf(last[:, 7]).all()
        last[:, [3, 5, 7]] = ref[:, n - 1, [3, 5, 7]]
        if b == 0:
            assert np.isposinf(got[:, :, 1]).all()
            got[:, :, 1] = ref[:, :, 1]
        assert rel_err_rms_floor(got, ref) <= 1e-5
    ctx.close()


# At most 16 rows, bf16, head dimension 128: the wavefronts of a workgroup split the keys - context lengths around a
# tile and around one and two rounds of eight tiles (heads that fill the chip), and the shapes that keep key splits.  P carries 16 mantissa bits (2^-17).
@pytest.mark.parametrize("N", [1, 5, 8, 16])
@pytest.mark.parametrize("q_scale,tol", [(1.0, 5e-5), (12.0, 3e-4)])
def test_attention_few_rows(pkg, N, q_scale, tol):
    for B, H, cap, ctx_len in [(1, 2, 8, [0]), (3, 2, 300, [1, 31, 33]), (1, 4, 2048, [2000]),
                               (5, 32, 600, [600, 0, 257, 31, 512]), (9, 15, 270, [270, 1, 64, 32, 255, 256, 65, 224, 223])]:
        print(f"attention few rows N={N} B={B} H={H} ctx={ctx_len} q_scale={q_scale}", flush=True)
        case = workloads.make_attention_case(N + B, B, H, N, 128, cap, ctx_len, "bf16", q_scale=q_scale)
        trees = _trees(N, B, N, 128, "chain" if N < 8 else "beam")
        n_nodes = np.array([t["n_nodes"] for t in trees], dtype=np.int32)
        q, kt, vt = case.q.copy(), case.k_tree.copy(), case.v_tree.copy()
        for b in range(B):
            q[b, :, n_nodes[b]:] = kt[b, :, n_nodes[b]:] = vt[b, :, n_nodes[b]:] = np.nan
        mask = torch.from_numpy(np.stack([t["anc_mask"] for t in trees]).view(np.int64)).cuda()
        ctx = pkg.Context(max_batch=B, max_slots=1, max_topk=1, max_vocab_rows=8, max_nodes=N, max_heads=H, max_head_dim=128)
        args = (to_device(q, "bf16"), to_device(case.k_cache, "bf16"), to_device(case.v_cache, "bf16"), dev_i64(case.kv_off),
                dev_i32(case.ctx_len), cap, to_device(kt, "bf16"), to_device(vt, "bf16"), dev_i32(n_nodes), mask, 128 ** -0.5)
        out, again = pkg.tree_verify_attn(ctx, *args).cpu().numpy(), pkg.tree_verify_attn(ctx, *args).cpu().numpy()
        for b in range(B):
            n = int(n_nodes[b])
            ref = oracle.tree_attention(case.q[b], case.k_cache[b], case.v_cache[b], int(case.ctx_len[b]), case.k_tree[b],
                                        case.v_tree[b], n, trees[b]["mask"], 128 ** -0.5)
            assert rel_err_rms_floor(out[b, :, :n], ref) <= tol
            assert np.array_equal(out[b, :, :n], again[b, :, :n])
        ctx.close()


# Caches whose capacity is past the last-level cache's size, with short histories: the same bits as the same rows in small caches.
@pytest.mark.parametrize("N", [8, 16, 17, 64])
def test_attention_large_capacity(pkg, N):
    B, H, big, small = 5, 32, 2600, 512  # 5 x 32 x 2600 x 512 bytes: 213 MB
    g = torch.Generator(device="cuda").manual_seed(N)
    rnd = lambda *shape: torch.randn(shape, generator=g, device="cuda").to(torch.bfloat16)
    q, kt, vt, ks, vs = rnd(B, H, N, 128), rnd(B, H, N, 128), rnd(B, H, N, 128), rnd(B, H, small, 128), rnd(B, H, small, 128)
    kb, vb = (torch.full((B, H, big, 128), float("nan"), device="cuda", dtype=torch.bfloat16) for _ in range(2))
    kb[:, :, :small], vb[:, :, :small] = ks, vs
    lens, nodes = dev_i32(np.array([512, 300, 511, 1, 0], dtype=np.int32)), dev_i32(np.array([N, 1, N, N // 2, N], dtype=np.int32))
    mask = torch.tensor([[-1 if i == 63 else (1 << (i + 1)) - 1] for i in range(N)], device="cuda").view(1, N, 1).repeat(B, 1, 1)
    outs = []
    for cap, k, v in ((big, kb, vb), (small, ks, vs)):
        ctx = pkg.Context(max_batch=B, max_slots=1, max_topk=1, max_vocab_rows=8, max_nodes=N, max_heads=H, max_head_dim=128)
        off = dev_i64(np.arange(B, dtype=np.int64) * H * cap * 128)
        out = torch.zeros((B, H, N, 128), device="cuda")
        outs.append(pkg.tree_verify_attn(ctx, q, k, v, off, lens, cap, kt, vt, nodes, mask, 0.09, out=out))
        torch.cuda.synchronize()
        ctx.close()
    assert torch.isfinite(outs[0]).all() and torch.equal(outs[0], outs[1])


# Histories that are past what stays in the last-level cache are read with streaming loads: the same bits as from calls for
# some of the sequences at a time, which read less (144 and 90 MB with 64 rows; 282 and 176 MB with 16 rows and fewer).
@pytest.mark.parametrize("N", [8, 16, 17, 64])
def test_attention_long_histories(pkg, N):
    B, H, L = 8, 32, 2150 if N <= 16 else 1100
    cap = L + 5
    g = torch.Generator(device="cuda").manual_seed(N)
    rnd = lambda *shape: torch.randn(shape, generator=g, device="cuda").to(torch.bfloat16)
    q, kt, vt, k, v = rnd(B, H, N, 128), rnd(B, H, N, 128), rnd(B, H, N, 128), rnd(B, H, cap, 128), rnd(B, H, cap, 128)
    lens = np.array([L, L - 1, L - 31, L, L - 32, L, L - 33, L], dtype=np.int32)
    mask = torch.tensor([[-1 if i == 63 else (1 << (i + 1)) - 1] for i in range(N)], device="cuda").view(1, N, 1).repeat(B, 1, 1)
    ctx = pkg.Context(max_batch=B, max_slots=1, max_topk=1, max_vocab_rows=8, max_nodes=N, max_heads=H, max_head_dim=128)

    def call(s):
        n = len(lens[s])
        off = dev_i64(np.arange(n, dtype=np.int64) * H * cap * 128)
        part = [x[s].contiguous() for x in (q, k, v, kt, vt, mask)]
        out = pkg.tree_verify_attn(ctx, *part[:3], off, dev_i32(lens[s]), cap, *part[3:5], dev_i32(np.full(n, N)), part[5], 0.09)
        torch.cuda.synchronize()
        return out

    whole = call(slice(0, 8))
    assert torch.isfinite(whole).all()
    assert torch.equal(whole[:5], call(slice(0, 5))) and torch.equal(whole[3:], call(slice(3, 8)))
    ctx.close()


# Few heads over a long capacity: eight key splits (bf16, 128) and more, which the merge takes eight at a time - all of them with keys,
# and with histories so short that most splits have none.  An infinity in the cache stays in its component (float and other
# head dimensions).
@pytest.mark.parametrize("dtype,dh,H,N,cap,tol", [("f32", 128, 2, 16, 2000, 1e-5), ("f32", 64, 1, 100, 2500, 1e-5),
                                                  ("bf16", 80, 1, 40, 3000, 1e-5), ("bf16", 128, 4, 64, 2048, 5e-5),
                                                  ("bf16", 128, 2, 128, 2048, 5e-5), ("bf16", 128, 3, 8, 2500, 5e-5)])
@pytest.mark.parametrize("short", [0, 1])
def test_attention_many_splits(pkg, dtype, dh, H, N, cap, tol, short):
    B, ctx_len = 1, [33 if short else cap - 7]
    print(f"attention many splits {dtype} dh={dh} H={H} N={N} ctx={ctx_len}", flush=True)
    case = workloads.make_attention_case(dh + N, B, H, N, dh, cap, ctx_len, dtype)
    trees = _trees(N, B, N, 128, "beam")
    n = int(trees[0]["n_nodes"])
    vc = case.v_cache.copy()
    planted = dtype == "f32" or dh != 128
    if planted:
        vc[0][:, 2, 1] = np.inf
    mask = torch.from_numpy(np.stack([t["anc_mask"] for t in trees]).view(np.int64)).cuda()
    ctx = pkg.Context(max_batch=B, max_slots=1, max_topk=1, max_vocab_rows=8, max_nodes=N, max_heads=H, max_head_dim=dh)
    args = (to_device(case.q, dtype), to_device(case.k_cache, dtype), to_device(vc, dtype), dev_i64(case.kv_off),
            dev_i32(case.ctx_len), cap, to_device(case.k_tree, dtype), to_device(case.v_tree, dtype), dev_i32(np.array([n])), mask,
            dh ** -0.5)
    got, again = pkg.tree_verify_attn(ctx, *args).cpu().numpy()[0, :, :n], pkg.tree_verify_attn(ctx, *args).cpu().numpy()[0, :, :n]
    ref = oracle.tree_attention(case.q[0], case.k_cache[0], case.v_cache[0], ctx_len[0], case.k_tree[0], case.v_tree[0], n,
                                trees[0]["mask"], dh ** -0.5)
    assert np.array_equal(got, again)
    if planted:
        assert np.isposinf(got[:, :, 1]).all()
        got[:, :, 1] = ref[:, :, 1]
    assert rel_err_rms_floor(got, ref) <= tol
    ctx.close()


# The draft head, the attention and the base head of one context on streams of their own, as the header allows: each has scratch of its own, so
# what runs beside a call changes none of its bits.
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_stages_on_three_streams(pkg, dtype):
    B, H, N, dh, cap, ctx_len, D, V, T, k = 2, 8, 64, 64, 1200, [1100, 900], 4096, 1500, 6, 4
    print(f"three streams {dtype}", flush=True)
    case = workloads.make_attention_case(3, B, H, N, dh, cap, ctx_len, dtype)
    trees = _trees(3, B, N, 128, "beam")
    n_nodes = dev_i32(np.array([t["n_nodes"] for t in trees]))
    mask = torch.from_numpy(np.stack([t["anc_mask"] for t in trees]).view(np.int64)).cuda()
    attn = (to_device(case.q, dtype), to_device(case.k_cache, dtype), to_device(case.v_cache, dtype), dev_i64(case.kv_off),
            dev_i32(case.ctx_len), cap, to_device(case.k_tree, dtype), to_device(case.v_tree, dtype), n_nodes, mask, dh ** -0.5)
    g = torch.Generator(device="cuda").manual_seed(3)
    h, hn, w = (torch.randn(s, generator=g, device="cuda").to(attn[0].dtype) for s in ((B, T, D), (B, N, D), (V, D)))
    ctx = pkg.Context(max_batch=B, max_slots=T, max_topk=k, max_vocab_rows=V, max_nodes=N, max_heads=H, max_head_dim=dh)
    stages = (lambda: pkg.ctc_draft_topk(ctx, h, w, None, k), lambda: {"out": pkg.tree_verify_attn(ctx, *attn)},
              lambda: pkg.verify_head_argmax(ctx, hn, w, n_nodes, want_logits=True))
    want = [stage() for stage in stages]
    torch.cuda.synchronize()
    streams, got = [torch.cuda.Stream() for _ in stages], []
    for _ in range(10):
        for stream, stage, ref in zip(streams, stages, want):
            with torch.cuda.stream(stream):
                ctx.set_stream(stream)
                got.append((stage(), ref))
    torch.cuda.synchronize()
    ctx.set_stream(torch.cuda.current_stream())
    live = torch.arange(N, device="cuda") < n_nodes[:, None]
    for res, ref in got:
        for name, t in ref.items():
            if t is None:
                continue
            a, b = (t, res[name]) if name != "out" else (t.transpose(1, 2)[live], res[name].transpose(1, 2)[live])
            assert torch.equal(a, b), name
    ctx.close()


# More than eight key splits (test_launch_plans.py asks the rule) whose maxima grow from one group of eight to the next: keys
# that some rows score far above the rest lie in tiles of the splits behind the first eight.  P carries 16 mantissa bits (2^-17) at
# bf16 and 128, 24 elsewhere; one sequence has keys in every split, the other in the first three only.
MORE_SPLITS = [("bf16", 128, 1, 8, 4096, 3e-4), ("bf16", 128, 1, 17, 16384, 3e-4), ("bf16", 128, 1, 100, 16384, 3e-4),
               ("bf16", 128, 2, 64, 16384, 3e-4), ("f32", 16, 2, 30, 4096, 1e-5), ("f32", 8, 1, 100, 6000, 1e-5),
               ("bf16", 64, 1, 40, 16384, 1e-5), ("f32", 128, 1, 64, 4096, 1e-5)]


@pytest.mark.parametrize("dtype,dh,H,N,cap,tol", MORE_SPLITS)
def test_attention_maxima_behind_eight_splits(pkg, dtype, dh, H, N, cap, tol):
    for ctx_len in (cap - 7, 70):
        print(f"attention maxima behind eight splits {dtype} dh={dh} H={H} N={N} ctx={ctx_len}", flush=True)
        case = workloads.make_attention_case(dh + N, 1, H, N, dh, cap, [ctx_len], dtype)
        trees = _trees(N, 1, N, 128, "beam")
        n = int(trees[0]["n_nodes"])
        kc = case.k_cache.copy()
        for row in range(0, n, 3):  # a key along that row's query, in the tile of split 8 + row / 3
            q = case.q[0, :, row]
            kc[0][:, 32 * (8 + row // 3 % 8) + row % 32] = workloads.round_to_storage(
                q * (20.0 * np.sqrt(dh) / np.square(q).sum(-1, keepdims=True)), dtype)
        mask = torch.from_numpy(np.stack([t["anc_mask"] for t in trees]).view(np.int64)).cuda()
        ctx = pkg.Context(max_batch=1, max_slots=1, max_topk=1, max_vocab_rows=8, max_nodes=N, max_heads=H, max_head_dim=dh)
        got = pkg.tree_verify_attn(ctx, to_device(case.q, dtype), to_device(kc, dtype), to_device(case.v_cache, dtype),
                                   dev_i64(case.kv_off), dev_i32(case.ctx_len), cap, to_device(case.k_tree, dtype),
                                   to_device(case.v_tree, dtype), dev_i32(np.array([n])), mask, dh ** -0.5).cpu().numpy()[0, :, :n]
        ref = oracle.tree_attention(case.q[0], kc[0], case.v_cache[0], ctx_len, case.k_tree[0], case.v_tree[0], n,
                                    trees[0]["mask"], dh ** -0.5)
        assert rel_err_rms_floor(got, ref) <= tol
        ctx.close()
