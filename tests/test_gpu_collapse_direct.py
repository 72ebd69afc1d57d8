"""ctc_collapse_tree where all raw candidates take part in one sort (k^T <= 512), around that limit, with tied scores,
a beam smaller and larger than the number of drafts, and a node cap."""
import numpy as np
import pytest
import torch

import workloads
from workloads.device import dev_f32, dev_i32
from test_gpu_parity import _run_stage3, _stage3_ctx

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pkg():
    import paper_2412_00061_amd as m
    return m


@pytest.mark.parametrize("T,k", [(3, 8), (8, 2), (5, 3), (4, 4), (2, 1), (6, 3)])
@pytest.mark.parametrize("quantum", [0.0, 0.5])
def test_collapse_direct(pkg, T, k, quantum):
    B, blank = 3, 40
    ctx = _stage3_ctx(pkg, B, T, k)
    for seed, vocab in ((1, max(k + 1, 5)), (2, 30)):
        ids, logp = workloads.make_topk_case(10 * T + seed, B, T, k, blank, vocab=vocab, p_blank=0.5, quantum=quantum)
        logp -= np.float32(1.0)  # log-probabilities below zero: the kernel's score keys hold no negative zero
        for beam, nodes in ((128, 128), (16, 128), (5, 9)):
            print(f"collapse T={T} k={k} quantum={quantum} beam={beam} nodes={nodes}", flush=True)
            _run_stage3(pkg, ctx, ids, logp, np.array([1, 2, 3]), blank, beam, nodes)
    ctx.close()


# A slot whose log-probabilities are no numbers (a hidden state that is none) leaves no draft and the root alone, whether
# all candidates take part in the sort (k^T <= 512) or a threshold picks them; -inf is an ordinary, worst value.
@pytest.mark.parametrize("T,k,slot", [(4, 2, 0), (4, 2, 3), (8, 2, 2), (5, 4, 0), (5, 4, 4)])
def test_scores_not_a_number(pkg, T, k, slot):
    B, blank, beam, nodes = 2, 40, 16, 64
    ctx = _stage3_ctx(pkg, B, T, k)
    ids, logp = workloads.make_topk_case(T + slot, B, T, k, blank, vocab=30, p_blank=0.3, quantum=0.0)
    logp -= np.float32(1.0)
    bad = logp.copy()
    bad[0, slot] = np.nan
    print(f"collapse T={T} k={k} NaN in slot {slot}", flush=True)
    got = pkg.ctc_collapse_tree(ctx, dev_i32(ids), dev_f32(bad), dev_i32(np.array([1, 2])), blank, beam, nodes)
    want = pkg.ctc_collapse_tree(ctx, dev_i32(ids), dev_f32(logp), dev_i32(np.array([1, 2])), blank, beam, nodes)
    assert int(got["n_cand"][0]) == 0 and int(got["n_nodes"][0]) == 1 and int(got["node_token"][0, 0]) == 1
    assert (got["cand_tokens"][0] == -1).all() and (got["node_token"][0, 1:] == -1).all()
    for name, v in want.items():
        assert torch.equal(got[name][1], v[1]), name
    low = logp.copy()
    low[:, slot, k - 1] = -np.inf
    _run_stage3(pkg, ctx, ids, low, np.array([1, 2]), blank, beam, nodes)
    ctx.close()
