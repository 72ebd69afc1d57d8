"""The launch rules, asked on the CPU (launch_plans.py): what they promise, and which kernels the GPU tests' sizes reach."""
import pytest

import launch_plans
import test_gpu_attn_any as attn_any
import test_gpu_attn_peaked as attn_peaked
import test_gpu_dma_tile as dma_tile
import test_gpu_head_shapes as head_shapes
import test_gpu_launch_modes as launch_modes
import test_zz_no_alloc as zz_no_alloc


def test_range_sums_fit_their_scratch():
    lines, rows_of = [], []
    for cols in (1, 8, 17, 40, 64, 128, 200, 512):
        for V in (1, 129, 1500, 5000, 9000, 16384, 16385):
            for D in (64, 1031, 4096):
                for f32 in (0, 1):
                    for what in ("b", "d") if cols <= 64 else ("b",):
                        lines.append((what, cols, D, V, f32, 4))
                        rows_of.append((V + 127) // 128 * 128)
    taken = 0
    for line, rows, (way, tile, ranges) in zip(lines, rows_of, launch_plans.ask(lines)):
        what, cols, D, V, f32, _ = line
        if way == "ranges":
            taken += 1
            steps = D * (4 if f32 else 2) // 256
            assert V <= 16384 and tile in (16, 32, 64, 128) and 1 <= ranges <= max(1, steps)
            assert ranges * cols * rows <= (2 if what == "d" else 4) << 20
    assert taken > 200


# A context keeps room by its limits: whatever fits them fits the room, which is a few KB where the limits are small.
def test_head_room_by_the_limits():
    _, draft, base = launch_plans.head_room(1, 8)
    assert draft == base == 16 * 128
    assert launch_plans.head_room(64, 32001)[1:] == (2 << 20, 4 << 20)  # (all that a call may leave)
    limits = [(c, r) for c in (1, 7, 40, 64, 200, 512) for r in (1, 128, 129, 1000, 5000, 16384, 40000)]
    rooms = launch_plans.ask([("s", c, r) for c, r in limits])
    for (cols, rows), (_, draft, base) in zip(limits, rooms):
        calls = [(w, max(1, c), D, max(1, V), f32, 8) for c in (cols, cols * 2 // 3) for V in (rows, rows // 2) for D in (256, 1031, 4096, 16384)
                 for f32 in (0, 1) for w in (("b", "d") if c <= 64 else ("b",))]
        for (w, c, D, V, f32, _), (way, _, ranges) in zip(calls, launch_plans.ask(calls)):
            assert way != "ranges" or ranges * c * ((V + 127) // 128 * 128) <= (draft if w == "d" else base)


@pytest.mark.parametrize("two_bf16", [0, 1])
def test_attention_splits_fit_their_scratch(two_bf16):
    lines = [("a", B, H, nodes, cap, dh, f32, two_bf16) for B in (1, 3, 8) for H in (1, 7, 32, 40) for nodes in (1, 16, 17, 64, 65, 128)
             for cap in (0, 40, 300, 2048, 20000) for dh, f32 in ((128, 0), (128, 1), (64, 0), (16, 1)) if not (two_bf16 and f32)]
    for (_, B, H, nodes, cap, dh, f32, _), (way, blocks, splits) in zip(lines, launch_plans.ask(lines)):
        units = max(256, B * H)  # of 128 query rows
        rows = 64 if way in ("any", "rows64") else 128
        assert blocks * rows >= nodes or way == "few"
        assert 1 <= splits <= 32 and (splits == 1 or B * H * blocks * splits * rows <= units * 128)


# As many splits as fill the chip stay where the model sees less than 3 % in another plan: shapes that got 13 % slower with a plan
# of the model's, and calls where the model's plan was 1.2 to 1.7 times as fast.
def test_attention_leaves_the_full_chip_only_for_a_clear_gain():
    assert launch_plans.attention(8, 14, 41, 381, 32, "f32") == ("any", 1, 4)
    assert launch_plans.attention(8, 12, 42, 840, 80, "f32") == ("any", 1, 5)
    assert launch_plans.attention(2, 40, 128, 144, 128, "bf16") == ("rows64", 2, 1)
    assert launch_plans.attention(6, 32, 128, 216, 128, "bf16") == ("rows128", 1, 1)
    assert launch_plans.attention(8, 26, 128, 845, 128, "bf16") == ("rows128", 1, 1)
    assert launch_plans.attention(3, 28, 128, 78, 128, "f32") == ("any", 2, 1)
    assert launch_plans.attention(1, 4, 128, 48, 16, "f32") == ("any", 2, 1)
    assert launch_plans.attention(1, 32, 128, 2064, 128, "bf16") == ("rows64", 2, 4)
    assert launch_plans.attention(1, 14, 35, 1939, 128, "f32")[2] > 8


# Heads whose columns a thread holds eight groups of rows of take their own kernels where the ranges measured slower; what gained
# takes the ranges.
def test_heads_of_many_rows_take_the_ranges_only_for_a_clear_gain():
    assert launch_plans.draft_head(18, 768, 10174, "f32", 3)[0] == "tile"
    assert launch_plans.draft_head(48, 772, 15938, "f32", 5)[0] == "tile"
    assert launch_plans.base_head(85, 2040, 9043, "bf16")[0] == "tile"
    assert launch_plans.draft_head(40, 3432, 10988, "bf16", 4)[0] == "ranges"
    assert launch_plans.draft_head(8, 4096, 4001, "bf16", 4)[0] == "ranges"
    assert launch_plans.draft_head(8, 4096, 8001, "bf16", 4)[0] == "stream"
    assert launch_plans.base_head(128, 4096, 6189, "bf16")[0] == "ranges"
    assert {launch_plans.base_head(c, 544, 68, "f32")[0] for c in (6, 32, 120, 256)} == {"ranges"}  # a lone float row block
    assert {launch_plans.base_head(c, 256, 68, "f32")[0] for c in (6, 32, 120, 512)} == {"tile"}


# ---- which kernels the GPU tests' sizes reach ---------------------------------------------------------------------------
def test_head_cases_take_the_kernels_they_are_meant_for():
    for B, T, D, Vp1, dtype, way in head_shapes.DRAFT_OWN_KERNEL:
        assert {launch_plans.draft_head(B * T, D, Vp1, dtype, k) for k in range(1, 9)} == {way}
    for B, N, D, V, dtype, way in head_shapes.BASE_WIDE:
        assert launch_plans.base_head(B * N, D, V, dtype) == way
    assert [launch_plans.draft_head(B * T, D, Vp1, dtype, k)[0] for B, T, D, Vp1, k, dtype in zz_no_alloc.SEQUENCE] == [
        "stream", "stream", "ranges", "stream", "tile", "stream", "tile", "ranges", "tile"]
    for way, (B, T, D, Vp1, k) in launch_modes.DEFERRED_HEADS.items():
        assert launch_plans.draft_head(B * T, D, Vp1, "bf16", k)[0] == way


def test_head_cases_take_the_loops_they_are_meant_for():
    for elem, dtype in ((2, "bf16"), (4, "f32")):
        for row in dma_tile.ROW_BYTES:
            for cols in (7, 32, 50, 128):
                assert launch_plans.base_head(cols, row // elem, 16500, dtype)[0] == "tile"
                assert launch_plans.head_loop(cols, row // elem, 16500, dtype)[0] == "dma"
            assert launch_plans.head_loop(200, row // elem, 16500, dtype)[:2] == ("dma", 128)
            assert {launch_plans.head_loop(cols, row // elem, 16500, dtype)[:2] for cols in (520, 732)} == {("dma", 256)}
            assert launch_plans.draft_head(21, row // elem, 16500, dtype, 4)[0] in ("tile", "stream")
    assert launch_plans.head_loop(200, 65, 16500, "bf16")[:2] == ("registers", 128)  # rows that start anywhere
    assert launch_plans.head_loop(50, 128, 16500, "bf16")[0] == "registers"  # rows of one step
    assert launch_plans.head_loop(50, 512, 128, "bf16")[0] == "registers"  # a single row block
    assert launch_plans.draft_head(64, 512, 128, "bf16", 4)[0] != "stream"


def test_cases_of_single_steps_have_them():
    for dtype, cols, D, V in dma_tile.SINGLE_STEPS:
        way, _, ranges = launch_plans.base_head(cols, D, V, dtype)
        assert launch_plans.head_loop(cols, D, V, dtype, ranges)[0] == "registers"
        assert way == "ranges" and ranges * 256 >= D * (4 if dtype == "f32" else 2)


def test_attention_cases_take_the_splits_they_are_meant_for():
    for dtype, dh, H, N, cap, _ in attn_any.MORE_SPLITS:
        assert launch_plans.attention(1, H, N, cap, dh, dtype)[2] >= 16
    got = {n: launch_plans.attention(B, H, N, cap, 128, "bf16") for n, (B, H, N, cap, _, _) in attn_peaked.SHAPES.items()}
    assert got == attn_peaked.TAKES
