"""The workloads by which this framework's speed is judged: what a serving or training program has it do.

Every case is one call, or one chain of calls, through the package's public entry points on inputs that are already on
the GPU.  The kinds of work:

  step        one decoding step as a serving loop issues it: draft head, CTC transform and token tree, verification
              attention, the base model's head, greedy acceptance, history update - in a row, issued
              through `prepared` calls as such loops do
  draft_head  the draft module's LM head with top-k, alone
  attention   one layer of the tree-masked verification attention, alone (a full model runs one per layer)
  base_head   the base model's head over all tree nodes, reduced to the greedy token
  sampled     the sampling form of it: the head with its logits, then the target's token drawn at every node
  draft_layer the draft module's transformer layer
  loss        the training objective and its gradient

Sizes are those of the workloads in `workloads/configs.py` (7B and 13B shapes, single sequences and a ragged batch of
eight, the tiny float32 shape), of the loss's two readings (thousands of positions with eight frames each; whole
sequences of up to 2048 frames), and generic smaller models in float32 and bfloat16.  `draw` spreads over the same ranges,
sizes that are no multiple of anything among them.
"""
import math

import torch

import paper_2412_00061_amd as pkg

BF16_7B = dict(D=4096, V=32000, T=8, k=4, H=32, dh=128, dtype="bf16")


def listed():
    return [
        # the smallest call: one step of the float32 shape that fits on a CPU; nothing but launches and latency
        dict(name="step_tiny_f32", kind="step", B=1, D=64, V=100, T=4, k=2, beam=16, nodes=128, H=4, dh=16,
             ctx_lo=32, ctx_hi=32, dtype="f32"),
        # the headline: interactive decoding of one sequence with a 7B model at 2048 cached positions
        dict(name="step_7b_ctx2048", kind="step", B=1, beam=128, nodes=128, ctx_lo=2048, ctx_hi=2048, **BF16_7B),
        # the draft head when eight sequences are decoded together: 64 columns on one pass over the weights
        dict(name="draft_head_7b_b8", kind="draft_head", B=8, T=8, D=4096, V=32000, k=4, dtype="bf16"),
        # a smaller model kept in float32 (parity runs, models that are not quantised to bf16)
        dict(name="draft_head_f32", kind="draft_head", B=2, T=8, D=2048, V=32000, k=4, dtype="f32"),
        # verification attention of a batch of eight sequences of 256 to 2048 cached positions (continuous batching)
        dict(name="attention_7b_b8_ragged", kind="attention", B=8, H=32, dh=128, nodes=64, ctx_lo=256, ctx_hi=2048,
             dtype="bf16"),
        # the attention of a small float32 model: head dimension 64, a tree that fills no whole block
        dict(name="attention_f32_dh64", kind="attention", B=2, H=12, dh=64, nodes=100, ctx_lo=300, ctx_hi=900,
             dtype="f32"),
        # the base model's head over the trees of eight sequences: 512 columns
        dict(name="base_head_7b_b8", kind="base_head", B=8, nodes=64, D=4096, V=32000, dtype="bf16"),
        # sampling-based acceptance of one sequence: the head writes its logits, one draw per node
        dict(name="sampled_7b", kind="sampled", B=1, nodes=128, D=4096, V=32000, temperature=0.8, dtype="bf16"),
        # the draft module's layer for one sequence and for a batch of eight (8 and 64 columns)
        dict(name="draft_layer_7b_b1", kind="draft_layer", B=1, T=8, D=4096, H=32, F=11008, ctx_lo=2048, ctx_hi=2048),
        dict(name="draft_layer_7b_b8", kind="draft_layer", B=8, T=8, D=4096, H=32, F=11008, ctx_lo=256, ctx_hi=2048),
        # training: thousands of positions, each with eight frames against the next tokens
        dict(name="loss_positions", kind="loss", B=2048, T=8, V=32000, Lmax=8),
        # training: whole padded sequences against long labels
        dict(name="loss_sequences", kind="loss", B=4, T=2048, V=32000, Lmax=1024),
    ]


# ---- drawn cases -------------------------------------------------------------------------------------------------
def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _hidden_size(rng, lo, hi):
    """Hidden sizes: mostly the multiples of 256 that models have, sometimes any multiple of 8, sometimes any number."""
    d = _log_int(rng, lo, hi)
    u = rng.random()
    if u < 0.6:
        return max(lo, (d + 128) // 256 * 256) if d >= 256 else (d + 31) // 32 * 32
    return (d + 7) // 8 * 8 if u < 0.85 else d


def _heads(rng, dtype):
    """(H, dh): 128 is the model family's head dimension, the others are what smaller models have."""
    dh = rng.choice([128, 128, 128, 64, 64, 96, 80] if dtype == "bf16" else [64, 64, 128, 16, 32, 80])
    return _log_int(rng, 4, 40 if dh == 128 else 32), dh


def draw(rng):
    kind = rng.choice(["step", "draft_head", "attention", "base_head", "sampled", "draft_layer", "loss"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    if kind == "step":
        B = rng.choice([1, 1, 2, 4, 8])
        T = rng.randint(3, 8)
        k = rng.choice([2, 3, 4])
        H, dh = _heads(rng, dtype)
        hi = _log_int(rng, 32, 2048)
        nodes = rng.choice([32, 64, 128, rng.randint(9, 128)])
        return dict(kind=kind, B=B, D=_hidden_size(rng, *((512, 5120) if dtype == "bf16" else (64, 1024))),
                    V=_log_int(rng, 100, 32000 if dtype == "bf16" else 8000), T=T, k=k, beam=rng.randint(8, 128),
                    nodes=min(nodes, 512 // B), H=H, dh=dh, ctx_lo=max(1, hi // rng.randint(1, 8)), ctx_hi=hi,
                    dtype=dtype)
    if kind == "draft_head":
        return dict(kind=kind, B=rng.randint(1, 8), T=rng.randint(1, 8),
                    D=_hidden_size(rng, *((512, 5120) if dtype == "bf16" else (256, 2048))),
                    V=_log_int(rng, 1000, 50000 if dtype == "bf16" else 32000), k=rng.randint(1, 8), dtype=dtype)
    if kind == "attention":
        H, dh = _heads(rng, dtype)
        hi = _log_int(rng, 32, 2048)
        return dict(kind=kind, B=rng.choice([1, 1, 2, 3, 4, 8]), H=H, dh=dh,
                    nodes=rng.choice([16, 32, 64, 128, rng.randint(1, 128)]),
                    ctx_lo=max(1, hi // rng.randint(1, 8)), ctx_hi=hi, dtype=dtype)
    if kind == "base_head":
        B = rng.choice([1, 1, 2, 4, 8])
        nodes = rng.choice([32, 64, 128, rng.randint(1, 128)])
        return dict(kind=kind, B=B, nodes=min(nodes, 512 // B),
                    D=_hidden_size(rng, *((512, 5120) if dtype == "bf16" else (256, 1024))),
                    V=_log_int(rng, 1000, 32000 if dtype == "bf16" else 8000), dtype=dtype)
    if kind == "sampled":
        return dict(kind=kind, B=rng.choice([1, 1, 2, 4]), nodes=rng.choice([32, 64, 128, rng.randint(1, 128)]),
                    D=_hidden_size(rng, *((512, 4096) if dtype == "bf16" else (256, 1024))),
                    V=_log_int(rng, 1000, 32000 if dtype == "bf16" else 8000),
                    temperature=round(rng.uniform(0.5, 1.5), 3), dtype=dtype)
    if kind == "draft_layer":
        H = rng.choice([8, 16, 32, 40])
        dh = 128 if H >= 32 else rng.choice([64, 128])
        return dict(kind=kind, B=rng.randint(1, 8), T=rng.randint(1, 8), D=H * dh, H=H,
                    F=256 * rng.randint(2 * H * dh // 256, 3 * H * dh // 256), ctx_lo=rng.randint(1, 256),
                    ctx_hi=_log_int(rng, 256, 2048))
    if rng.random() < 0.5:
        T = rng.randint(4, 16)
        return dict(kind=kind, B=_log_int(rng, 64, 1024), T=T, V=_log_int(rng, 500, 32000), Lmax=rng.randint(1, T))
    T = _log_int(rng, 64, 2048)
    return dict(kind=kind, B=rng.randint(1, 4), T=T, V=_log_int(rng, 500, 32000), Lmax=max(1, T // rng.randint(2, 8)))


# ---- inputs ------------------------------------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _dtype(case):
    return torch.bfloat16 if case.get("dtype", "bf16") == "bf16" else torch.float32


def _randn(g, shape, dtype, scale=1.0):
    x = torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)
    return (x * scale if scale != 1.0 else x).to(dtype)


def _i32(g, lo, hi, shape):
    """Uniform in [lo, hi]."""
    return torch.randint(lo, hi + 1, shape, generator=g, device="cuda", dtype=torch.int32)


def _context(case, **more):
    lim = dict(max_batch=case.get("B", 1), max_slots=case.get("T", 8), max_topk=case.get("k", 4),
               max_vocab_rows=case.get("V", 1000) + 1, max_nodes=case.get("nodes", 64), max_heads=case.get("H", 1),
               max_head_dim=case.get("dh", 128))
    lim.update(more)
    return pkg.Context(**lim)


def _head_inputs(case, g):
    """Draft-head operands with the posteriors of a trained CTC head: the states of a sequence's slots are blends of a few
    head rows that neighbouring slots share, and the blank is a likely symbol - repeats and blanks occur in the lists."""
    B, T, D, V, dt = case["B"], case["T"], case["D"], case["V"], _dtype(case)
    w = _randn(g, (V + 1, D), dt, 0.02)
    tok = torch.randint(0, V, (B, T, 3), generator=g, device="cuda")
    same = torch.rand((B, T), generator=g, device="cuda") < 0.5
    for t in range(1, T):
        tok[:, t, 0] = torch.where(same[:, t], tok[:, t - 1, 0], tok[:, t, 0])
    coef = torch.tensor([1.0, 0.8, 0.65], device="cuda").view(1, 1, 3, 1)
    blend = (w[tok].float() * coef).sum(2)
    blend = blend / blend.square().mean(-1, keepdim=True).sqrt()
    noise = torch.randn((B, T, D), generator=g, device="cuda")
    hidden = 0.22 * blend + 0.975 * noise
    hidden = (hidden / hidden.square().mean(-1, keepdim=True).sqrt()).to(dt)
    bias = torch.zeros(V + 1, device="cuda")
    bias[V] = 3.0
    return hidden, w, bias


def _kv_inputs(case, g):
    """Attention operands: unit-scale queries, keys and values, ragged context lengths, one cache block per sequence."""
    B, H, dh, N, dt = case["B"], case["H"], case["dh"], case["nodes"], _dtype(case)
    cap = case["ctx_hi"] + 16
    kv = {n: _randn(g, (B, H, N, dh), dt) for n in ("q", "k_tree", "v_tree")}
    kv.update({n: _randn(g, (B, H, cap, dh), dt) for n in ("k_cache", "v_cache")})
    kv["ctx_len"] = _i32(g, case["ctx_lo"], case["ctx_hi"], (B,))
    kv["kv_off"] = torch.arange(B, device="cuda", dtype=torch.int64) * (H * cap * dh)
    kv["kv_cap"] = cap
    return kv


def _tree_mask(parent, n_nodes, N):
    """Ancestor masks (bit j of row i: node j is on the path root..i) of trees given by parents [B][N]."""
    words = (N + 63) // 64
    B = len(parent)
    mask = torch.zeros((B, N, words), dtype=torch.int64)
    for b in range(B):
        rows = []
        for i in range(n_nodes[b]):
            bits = 1 << i
            if i:
                bits |= rows[parent[b][i]]
            rows.append(bits)
            for wd in range(words):
                v = (bits >> (64 * wd)) & 0xFFFFFFFFFFFFFFFF
                mask[b, i, wd] = v - (1 << 64) if v >= (1 << 63) else v
    return mask


def _random_trees(case, seed):
    """Trees as the CTC transform builds them: at most 8 deep, breadth near the root, node ids in creation order."""
    rng = torch.Generator().manual_seed(int(seed))
    B, N = case["B"], case["nodes"]
    parents, counts = [], []
    for _ in range(B):
        n = N if N < 8 else int(torch.randint(3 * N // 4, N + 1, (1,), generator=rng))
        u = torch.rand(N, generator=rng).tolist()
        par, depth = [-1], [0]
        for i in range(1, n):
            j = int(u[i] * i)
            while depth[j] >= 8:
                j = par[j]
            par.append(j)
            depth.append(depth[j] + 1)
        parents.append(par)
        counts.append(n)
    return _tree_mask(parents, counts, N).cuda(), torch.tensor(counts, dtype=torch.int32, device="cuda")


def _zeros(shape, dtype=torch.float32):
    return torch.zeros(shape, dtype=dtype, device="cuda")


def _prepare_step(case, g):
    B, T, k, D, V, N, H, dh, beam = (case[n] for n in ("B", "T", "k", "D", "V", "nodes", "H", "dh", "beam"))
    dt = _dtype(case)
    i32, code = torch.int32, (pkg.binding.CTCSPEC_BF16 if dt == torch.bfloat16 else pkg.binding.CTCSPEC_F32)
    ctx = _context(case)
    hidden, w, bias = _head_inputs(case, g)
    kv = _kv_inputs(case, g)
    root = _i32(g, 0, V - 1, (B,))
    node_hidden = _randn(g, (B, N, D), dt)
    w_base = _randn(g, (V, D), dt, 0.02)
    o = {
        "topk_id": _zeros((B, T, k), i32), "topk_logp": _zeros((B, T, k)), "lse": _zeros((B, T)),
        "logits": _zeros((B, T, V + 1)), "n_cand": _zeros((B,), i32), "cand_tokens": _zeros((B, beam, T), i32),
        "cand_len": _zeros((B, beam), i32), "cand_score": _zeros((B, beam)), "cand_leaf": _zeros((B, beam), i32),
        "n_nodes": _zeros((B,), i32), "node_token": _zeros((B, N), i32), "node_parent": _zeros((B, N), i32),
        "node_depth": _zeros((B, N), i32), "anc_mask": _zeros((B, N, (N + 63) // 64), torch.int64),
        "attention": _zeros((B, H, N, dh)), "target_argmax": _zeros((B, N), i32), "accept_len": _zeros((B,), i32),
        "accept_nodes": _zeros((B, T + 1), i32), "accept_tokens": _zeros((B, T + 1), i32), "next_token": _zeros((B,), i32),
        "ctx_len": _zeros((B,), i32), "k_cache": kv["k_cache"], "v_cache": kv["v_cache"],
    }
    tree = [o[n] for n in ("n_cand", "cand_tokens", "cand_len", "cand_score", "cand_leaf", "n_nodes", "node_token",
                           "node_parent", "node_depth", "anc_mask")]
    calls = [
        pkg.prepared(ctx, "ctc_draft_topk", code, hidden, w, bias, B, T, D, V + 1, k, o["topk_id"], o["topk_logp"],
                     o["lse"], o["logits"]),
        pkg.prepared(ctx, "ctc_collapse_tree", o["topk_id"], o["topk_logp"], root, B, T, k, V, beam, N, *tree),
        pkg.prepared(ctx, "tree_verify_attn", code, kv["q"], kv["k_cache"], kv["v_cache"], kv["kv_off"], kv["ctx_len"],
                     kv["kv_cap"], kv["k_tree"], kv["v_tree"], o["n_nodes"], o["anc_mask"], B, H, dh, N,
                     1.0 / math.sqrt(dh), o["attention"]),
        pkg.prepared(ctx, "verify_head_argmax", code, node_hidden, w_base, o["n_nodes"], B, N, D, V, o["target_argmax"],
                     None),
        pkg.prepared(ctx, "accept_longest", o["n_nodes"], o["node_token"], o["node_parent"], o["node_depth"],
                     o["target_argmax"], B, T, N, o["accept_len"], o["accept_nodes"], o["accept_tokens"], o["next_token"]),
        pkg.prepared(ctx, "kv_commit", code, kv["k_tree"], kv["v_tree"], o["accept_len"], o["accept_nodes"], T,
                     kv["kv_off"], kv["ctx_len"], kv["kv_cap"], B, H, dh, N, kv["k_cache"], kv["v_cache"], o["ctx_len"]),
    ]
    return dict(calls=calls, out=o, hidden=hidden, w=w, bias=bias, kv=kv, ctx=ctx)


def _prepare_layer(case, g):
    B, T, D, H, F = (case[n] for n in ("B", "T", "D", "H", "F"))
    dh, bf = D // H, torch.bfloat16
    cap = case["ctx_hi"] + 16
    w = {
        "ln1": (1.0 + 0.1 * torch.randn(D, generator=g, device="cuda")).to(bf),
        "wqkv": _randn(g, (3 * D, D), bf, 1.0 / math.sqrt(D)), "wo": _randn(g, (D, D), bf, 1.0 / math.sqrt(D)),
        "ln2": (1.0 + 0.1 * torch.randn(D, generator=g, device="cuda")).to(bf),
        "wgu": _randn(g, (2 * F, D), bf, 1.0 / math.sqrt(D)), "wd": _randn(g, (D, F), bf, 1.0 / math.sqrt(F)),
    }
    x = torch.randn((B, T, D), generator=g, device="cuda")
    # a few channels are much larger, as in a trained model's last layer
    x[..., torch.randint(0, D, (max(1, D // 256),), generator=g, device="cuda")] *= 8.0
    ctx_len = _i32(g, case["ctx_lo"], case["ctx_hi"], (B,))
    return dict(
        ctx=_context(case, max_nodes=max(8, T), max_head_dim=dh), x=x.to(bf), w=w,
        weights=pkg.layer_weights(**w), pos0=ctx_len.clone(),
        ctx_len=ctx_len, kv_off=torch.arange(B, device="cuda", dtype=torch.int64) * (H * cap * dh), kv_cap=cap,
        k_cache=_randn(g, (B, H, cap, dh), bf), v_cache=_randn(g, (B, H, cap, dh), bf),
        workspace=torch.empty(pkg.draft_layer_workspace_bytes(B, T, D, H, F), dtype=torch.uint8, device="cuda"),
        out={"out": _zeros((B, T, D), bf), "k_new": _zeros((B, H, T, dh), bf), "v_new": _zeros((B, H, T, dh), bf)})


def _prepare_loss(case, g):
    B, T, V, Lmax = (case[n] for n in ("B", "T", "V", "Lmax"))
    frame_len = _i32(g, max(1, 3 * T // 4), T, (B,))
    label_len = torch.minimum(_i32(g, Lmax // 2, Lmax, (B,)), frame_len)
    labels = _i32(g, 0, V - 1, (B, Lmax))
    logits = torch.randn((B, T, V + 1), generator=g, device="cuda")
    logits *= 2.0
    return dict(ctx=_context(case, max_batch=1, max_slots=1), logits=logits, labels=labels, label_len=label_len,
                frame_len=frame_len,
                workspace=torch.empty(pkg.ctc_loss_workspace_bytes(B, T, Lmax), dtype=torch.uint8, device="cuda"),
                out={"loss": _zeros((B,)), "grad": torch.empty((B, T, V + 1), device="cuda")})


def prepare(case, seed):
    g, kind = _gen(seed), case["kind"]
    if kind == "step":
        s = _prepare_step(case, g)
    elif kind == "draft_head":
        hidden, w, bias = _head_inputs(case, g)
        B, T, k = case["B"], case["T"], case["k"]
        s = dict(ctx=_context(case, max_topk=8), hidden=hidden, w=w, bias=bias,
                 out={"topk_id": _zeros((B, T, k), torch.int32), "topk_logp": _zeros((B, T, k)), "lse": _zeros((B, T))})
    elif kind == "attention":
        kv = _kv_inputs(case, g)
        mask, n_nodes = _random_trees(case, seed)
        s = dict(ctx=_context(case), kv=kv, mask=mask, n_nodes=n_nodes,
                 out={"out": _zeros((case["B"], case["H"], case["nodes"], case["dh"]))})
    elif kind in ("base_head", "sampled"):
        B, N, D, V = case["B"], case["nodes"], case["D"], case["V"]
        s = dict(ctx=_context(case), hidden=_randn(g, (B, N, D), _dtype(case)), w=_randn(g, (V, D), _dtype(case), 0.02),
                 n_nodes=_i32(g, max(1, 3 * N // 4), N, (B,)),
                 out={"target_argmax": _zeros((B, N), torch.int32)})
        if kind == "sampled":
            s["out"]["logits"] = _zeros((B, N, V))
            s["out"]["target_sampled"] = _zeros((B, N), torch.int32)
            s["uniforms"] = torch.rand((B, N), generator=g, device="cuda")
    elif kind == "draft_layer":
        s = _prepare_layer(case, g)
    else:
        s = _prepare_loss(case, g)
    s["case"] = case
    return s


def run(state):
    s, case = state, state["case"]
    kind = case["kind"]
    if kind == "step":
        for call in s["calls"]:
            call()
        return s["out"]
    if kind == "draft_head":
        return pkg.ctc_draft_topk(s["ctx"], s["hidden"], s["w"], s["bias"], case["k"], out=s["out"])
    if kind == "attention":
        kv = s["kv"]
        return pkg.tree_verify_attn(s["ctx"], kv["q"], kv["k_cache"], kv["v_cache"], kv["kv_off"], kv["ctx_len"],
                                    kv["kv_cap"], kv["k_tree"], kv["v_tree"], s["n_nodes"], s["mask"],
                                    1.0 / math.sqrt(case["dh"]), out=s["out"]["out"])
    if kind == "base_head":
        return pkg.verify_head_argmax(s["ctx"], s["hidden"], s["w"], s["n_nodes"], out=s["out"])
    if kind == "sampled":
        head = pkg.verify_head_argmax(s["ctx"], s["hidden"], s["w"], s["n_nodes"], want_logits=True, out=s["out"])
        drawn = pkg.verify_sample_tokens(s["ctx"], head["logits"], s["n_nodes"], s["uniforms"], case["temperature"],
                                         out=s["out"])
        return {**head, "target_sampled": drawn}
    if kind == "draft_layer":
        return pkg.draft_layer_forward(s["ctx"], s["x"], s["weights"], s["pos0"], s["k_cache"], s["v_cache"], s["kv_off"],
                                       s["ctx_len"], s["kv_cap"], case["H"], case["F"], 1e-6, 10000.0,
                                       workspace=s["workspace"], out=s["out"])
    return pkg.ctc_loss(s["ctx"], s["logits"], s["labels"], s["label_len"], s["frame_len"], case["V"],
                        workspace=s["workspace"], out=s["out"])


# ---- what a pass cannot do without -------------------------------------------------------------------------------
def _mean_ctx(case):
    return 0.5 * (case["ctx_lo"] + case["ctx_hi"])


def _attention_work(B, H, dh, N, ctx, e):
    return {"bytes": B * H * dh * (2 * e * (ctx + N) + N * (e + 4)), "flops": 4.0 * B * H * N * dh * (ctx + N)}


def _head_work(cols, D, V, e):
    return {"bytes": e * D * (V + cols), "flops": 2.0 * cols * D * V}


def work(case):
    kind = case["kind"]
    e = 4 if case.get("dtype", "bf16") == "f32" else 2
    parts = []
    if kind in ("step", "draft_head"):
        parts.append(_head_work(case["B"] * case["T"], case["D"], case["V"] + 1, e))
    if kind in ("step", "attention"):
        parts.append(_attention_work(case["B"], case["H"], case["dh"], case["nodes"], _mean_ctx(case), e))
    if kind in ("step", "base_head", "sampled"):
        parts.append(_head_work(case["B"] * case["nodes"], case["D"], case["V"], e))
    if kind == "step":
        parts.append({"bytes": 4.0 * case["B"] * case["T"] * (case["V"] + 1), "flops": 0.0})
    if kind == "sampled":  # the logits are part of the answer: written once (the draw need not read them again)
        parts.append({"bytes": 4.0 * case["B"] * case["nodes"] * case["V"], "flops": 0.0})
    if kind == "draft_layer":
        B, T, D, F = case["B"], case["T"], case["D"], case["F"]
        weights = 4 * D * D + 3 * D * F
        parts.append({"bytes": 2.0 * weights + 2.0 * B * T * D * 4, "flops": 2.0 * B * T * weights})
        parts.append(_attention_work(B, case["H"], D // case["H"], T, _mean_ctx(case), 2))
    if kind == "loss":
        n = case["B"] * case["T"]
        parts.append({"bytes": 8.0 * n * (case["V"] + 1),
                      "flops": 4.0 * n * (case["V"] + 1) + 20.0 * n * (2 * case["Lmax"] + 1)})
    return {"bytes": sum(p["bytes"] for p in parts), "flops": sum(p["flops"] for p in parts)}


def tolerance(case):
    """What another correct implementation at the same precision may differ by: sums of float32 numbers in another order
    (the bf16 operands' products are exact in float32), the probabilities of the bf16 attention at 16 mantissa bits,
    the bf16 rounding of the layer's queries, keys, values and output, and per call a handful of flipped ties."""
    kind = case["kind"]
    if kind == "draft_layer":
        return {"rel": 7e-3, "max": 0.05}
    if kind in ("loss", "attention", "step"):
        return {"rel": 2e-5, "max": 1e-3, "differ": 0.01}
    return {"rel": 1e-5, "max": 4e-4, "differ": 0.01}


# ---- the same outputs in 64 bits ---------------------------------------------------------------------------------
def _exact_head(hidden, w, bias, k):
    z = hidden.reshape(-1, hidden.shape[-1]).double() @ w.double().t()
    if bias is not None:
        z += bias.double()
    lse = torch.logsumexp(z, -1)
    top = torch.topk(z, k, -1).values - lse[:, None]
    B, T = hidden.shape[:2]
    return z.view(B, T, -1), top.view(B, T, k), lse.view(B, T)


def _exact_attention(q, k_cache, v_cache, ctx_len, k_tree, v_tree, n_nodes, mask, scale):
    """Rows beyond a sequence's nodes are left at zero."""
    B, H, N, dh = q.shape
    out = torch.zeros((B, H, N, dh), dtype=torch.float64, device=q.device)
    bit = torch.arange(64, device=q.device)
    for b in range(B):
        L, n = int(ctx_len[b]), int(n_nodes[b])
        keys = torch.cat([k_cache[b, :, :L], k_tree[b, :, :n]], 1).double()
        vals = torch.cat([v_cache[b, :, :L], v_tree[b, :, :n]], 1).double()
        seen = ((mask[b, :n, :, None] >> bit) & 1).bool().reshape(n, -1)[:, :n]
        s = (q[b, :, :n].double() @ keys.transpose(1, 2).contiguous()) * scale
        s[:, :, L:].masked_fill_(~seen[None], -math.inf)
        out[b, :, :n] = torch.softmax(s, -1) @ vals
    return out


def _exact_layer(s, case):
    B, T, D, H, F = (case[n] for n in ("B", "T", "D", "H", "F"))
    dh = D // H
    w = {n: t.double() for n, t in s["w"].items()}
    x = s["x"].double()

    def norm(y, gain):
        return y / torch.sqrt(y.square().mean(-1, keepdim=True) + 1e-6) * gain

    q, k, v = (norm(x, w["ln1"]) @ w["wqkv"].t()).view(B, T, 3, H, dh).permute(2, 0, 3, 1, 4)
    pos = (s["pos0"].view(B, 1).double() + torch.arange(T, device="cuda")).view(B, 1, T, 1)
    ang = pos * 10000.0 ** (-2.0 * torch.arange(dh // 2, device="cuda", dtype=torch.float64) / dh)

    def turn(y):
        a, c = y[..., : dh // 2], y[..., dh // 2:]
        return torch.cat([a * ang.cos() - c * ang.sin(), c * ang.cos() + a * ang.sin()], -1)

    q, k, v = turn(q), turn(k).contiguous(), v.contiguous()
    causal = torch.tensor([(2 << t) - 1 for t in range(T)], device="cuda").view(1, T, 1).expand(B, T, 1)
    a = _exact_attention(q, s["k_cache"], s["v_cache"], s["ctx_len"], k, v, torch.full((B,), T), causal, dh ** -0.5)
    h = x + a.permute(0, 2, 1, 3).reshape(B, T, D) @ w["wo"].t()
    gu = norm(h, w["ln2"]) @ w["wgu"].t()
    out = h + (torch.nn.functional.silu(gu[..., :F]) * gu[..., F:]) @ w["wd"].t()
    return {"out": out, "k_new": k, "v_new": v}


def _exact_loss(s, case):
    z = s["logits"].double().requires_grad_(True)
    logp = torch.log_softmax(z, -1).transpose(0, 1)
    args = (s["labels"].long(), s["frame_len"].long(), s["label_len"].long())
    loss = torch.nn.functional.ctc_loss(logp, *args, blank=case["V"], reduction="none", zero_infinity=False)
    with torch.no_grad():
        fits = torch.isfinite(loss)
    safe = torch.nn.functional.ctc_loss(logp, *args, blank=case["V"], reduction="none", zero_infinity=True)
    grad, = torch.autograd.grad((safe * fits).sum(), z)
    return {"loss": loss.detach(), "grad": grad}


def exact(case, seed):
    kind = case["kind"]
    s = prepare(case, seed)
    if kind == "step":
        z, top, lse = _exact_head(s["hidden"], s["w"], s["bias"], case["k"])
        # what follows depends on the tokens that were chosen; the attention alone is a kind of its own
        return {n: {"logits": z, "topk_logp": top, "lse": lse}.get(n) for n in s["out"]}
    if kind == "draft_head":
        _, top, lse = _exact_head(s["hidden"], s["w"], s["bias"], case["k"])
        return {"topk_id": None, "topk_logp": top, "lse": lse}
    if kind == "attention":
        kv = s["kv"]
        return _exact_attention(kv["q"], kv["k_cache"], kv["v_cache"], kv["ctx_len"], kv["k_tree"], kv["v_tree"],
                                s["n_nodes"], s["mask"], 1.0 / math.sqrt(case["dh"]))
    if kind in ("base_head", "sampled"):
        if kind == "base_head":
            return None  # whole numbers only
        z = s["hidden"].reshape(-1, case["D"]).double() @ s["w"].double().t()
        return {"target_argmax": None, "logits": z.view(case["B"], case["nodes"], -1), "target_sampled": None}
    if kind == "draft_layer":
        return _exact_layer(s, case)
    return _exact_loss(s, case)
