"""The draft layer's plan (csrc/layer_plan.h, host code), asked on the CPU: which workgroup shapes the GPU cases take, and
that the workspace which callers are told to bring holds what every smaller call needs."""
import os
import subprocess

import pytest

import paper_2412_00061_amd as pkg
from test_gpu_draft_layer import SHORT_RANGE_CASES, WIDE_CASES

CSRC = os.path.join(os.path.dirname(os.path.abspath(pkg.__file__)), "csrc")
CUS = 256  # compute units of the GPU
PROGRAM = r"""
#include <stdio.h>
#include "head_plan.h"
#include "layer_plan.h"
using namespace ctcspec;
int main() {
  char what;
  int a, b, c, d, e, f;
  while (scanf(" %c %d %d %d %d %d %d", &what, &a, &b, &c, &d, &e, &f) == 7) {
    LayerPlan pl;
    if (what == 'p') printf("%d\n", make_plan(pl, a, b, c, d, e) ? tile_columns(c) * 1000 + pl.rows : 0);
    else if (what == 't') printf("%d\n", make_plan(pl, a, b, c, c, d) && through_registers(pl, streamed_weights(2LL * (4LL * e * e + 3LL * e * f), 2LL * b)));
    else printf("%zu\n", layer_workspace(a, b, c, d, e, f, what == 'q').total);
  }
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    at = tmp_path_factory.mktemp("layer_plan")
    (at / "plan.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(at / "plan.cpp"), "-o", str(at / "plan")], check=True)

    def run(lines):
        text = "\n".join(" ".join(map(str, l)) for l in lines)
        return [int(x) for x in subprocess.run([str(at / "plan")], input=text, capture_output=True, text=True, check=True).stdout.split()]

    return run


def test_gpu_cases_take_every_workgroup_shape(ask):
    shapes = {tile * 1000 + rows for tile in (32, 64, 128) for rows in (128, 192, 256)} - {32 * 1000 + 192}
    lines = [("p", N, K, B * T, B * T, CUS, 0) for _, B, T, D, _, F, _, _ in WIDE_CASES
             for N, K in ((3 * D, D), (D, D), (2 * F, D), (D, F))]
    assert set(ask(lines)) == shapes


def test_ranges_that_go_through_registers(ask):
    def passes(B, T, D, F):
        return ask([("t", N, K, B * T, CUS, D, F) for N, K in ((3 * D, D), (D, D), (2 * F, D), (D, F))])

    for _, B, T, D, _, F, _, _ in SHORT_RANGE_CASES:
        assert passes(B, T, D, F)[0] == 1
    assert passes(1, 8, 4096, 11008) == [0, 1, 0, 0]
    assert passes(2, 8, 2048, 4096) == [1, 0, 1, 0]  # the others' ranges are of one trip
    assert passes(1, 8, 1024, 3072) == [0, 0, 0, 0]  # weights that may be cached
    assert passes(4, 8, 2048, 4096) == [0, 0, 0, 0]  # more than 16 columns


@pytest.mark.parametrize("D,H,F", [(256, 2, 512), (2048, 16, 5632), (4096, 32, 11008), (5120, 40, 13824)])
def test_workspace_holds_every_smaller_call(ask, D, H, F):
    sizes = [(B, T) for B in range(1, 13) for T in range(1, 65)]
    told = dict(zip(sizes, ask([("q", B, T, D, H, F, CUS) for B, T in sizes])))
    needed = dict(zip(sizes, ask([("n", B, T, D, H, F, CUS) for B, T in sizes])))
    assert all(needed[s] <= told[s] for s in sizes)  # (and what is told never falls: test_workspace_sizes.py)
