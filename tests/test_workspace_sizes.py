"""Workspaces sized for the largest shape serve every smaller one: the byte counts never fall as a size grows."""
import pytest

import paper_2412_00061_amd as pkg


@pytest.mark.parametrize("D,H,F", [(256, 2, 512), (2048, 16, 5632), (4096, 32, 11008), (5120, 40, 13824)])
def test_draft_layer_workspace_grows(D, H, F):
    table = [[pkg.draft_layer_workspace_bytes(B, T, D, H, F) for T in range(1, 65)] for B in range(1, 13)]
    for B, row in enumerate(table):
        assert all(row[i] <= row[i + 1] for i in range(len(row) - 1)), B + 1
        assert B == 0 or all(a <= b for a, b in zip(table[B - 1], row)), B + 1


@pytest.mark.parametrize("T", [1, 8, 63, 64, 65, 300])
def test_ctc_loss_workspace_grows(T):
    sizes = [1, 2, 17, 20, 62, 63, 64, 65, 127, 128, 1024, 2047]
    last = {}
    for B in [1, 2, 8, 400, 767, 768, 769, 800, 1000, 2000, 65535]:
        row = [pkg.ctc_loss_workspace_bytes(B, T, L) for L in sizes]
        assert row == sorted(row), B
        longer = [pkg.ctc_loss_workspace_bytes(B, T + 1, L) for L in sizes]
        assert all(a <= b for a, b in zip(row, longer)), B
        assert not last or all(a <= b for a, b in zip(last["row"], row)), B
        last["row"] = row
