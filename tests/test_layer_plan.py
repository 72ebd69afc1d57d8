"""The draft layer's plan (csrc/layer_plan.h, host code), asked on the CPU: which workgroup shapes the GPU cases take, and
that the workspace which callers are told to bring holds what every smaller call needs."""
import os
import subprocess

import pytest

import paper_2412_00061_amd as pkg
from test_gpu_draft_layer import WIDE_CASES

CSRC = os.path.join(os.path.dirname(os.path.abspath(pkg.__file__)), "csrc")
CUS = 256  # compute units of the GPU
PROGRAM = r"""
#include <stdio.h>
#include "layer_plan.h"
using namespace ctcspec;
int main() {
  char what;
  int a, b, c, d, e, f;
  while (scanf(" %c %d %d %d %d %d %d", &what, &a, &b, &c, &d, &e, &f) == 7) {
    LayerPlan pl;
    if (what == 'p') printf("%d\n", make_plan(pl, a, b, c, d, e) ? tile_columns(c) * 1000 + pl.rows : 0);
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


@pytest.mark.parametrize("D,H,F", [(256, 2, 512), (2048, 16, 5632), (4096, 32, 11008), (5120, 40, 13824)])
def test_workspace_holds_every_smaller_call(ask, D, H, F):
    sizes = [(B, T) for B in range(1, 13) for T in range(1, 65)]
    told = dict(zip(sizes, ask([("q", B, T, D, H, F, CUS) for B, T in sizes])))
    needed = dict(zip(sizes, ask([("n", B, T, D, H, F, CUS) for B, T in sizes])))
    assert all(needed[s] <= told[s] for s in sizes)  # (and what is told never falls: test_workspace_sizes.py)
