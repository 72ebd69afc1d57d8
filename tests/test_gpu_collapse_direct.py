"""ctc_collapse_tree where all raw candidates take part in one sort (k^T <= 512), around that limit, with tied scores,
a beam smaller and larger than the number of drafts, and a node cap."""
import numpy as np
import pytest

import workloads
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
