"""Asks the library's launch rules (csrc/head_plan.h, csrc/attn_plan.h: host code without HIP) which way a call takes, so
that a test can tell whether its sizes still reach the kernel that they were chosen for."""
import functools
import os
import subprocess
import tempfile

import paper_2412_00061_amd as pkg

CSRC = os.path.join(os.path.dirname(os.path.abspath(pkg.__file__)), "csrc")
PROGRAM = r"""
#include <stdio.h>
#include "attn_plan.h"
#include "head_plan.h"
using namespace ctcspec;
int main() {
  char what;
  int a, b, c, d, e, f, g;
  while (scanf(" %c %d %d %d %d %d %d %d", &what, &a, &b, &c, &d, &e, &f, &g) == 8) {
    HeadPlan p;
    p.cols = a; p.D = b; p.V = c;
    AttnShape s = {0, 0};
    if (what == 'd') {  // cols D V f32 k
      if (plan_draft_head(p, d != 0, e)) printf("ranges %d %d\n", p.tile_cols, p.splits);
      else if (!d && draft_stream_stages(a, b, c)) printf("stream %d %d\n", (a + 15) / 16, draft_stream_stages(a, b, c));
      else printf("tile %d 0\n", head_tile_cols(a) > 64 ? 64 : head_tile_cols(a));
    } else if (what == 'b') {  // cols D V f32
      if (plan_base_head(p, d != 0)) printf("ranges %d %d\n", p.tile_cols, p.splits);
      else printf("tile %d %d\n", head_tile_cols(a), a > kHeadColBlock ? 256 : 128);
    } else if (what == 'l') {  // cols D V f32 ranges
      const bool dma = dma_rows(c, b, d ? 4 : 2, e);
      printf("%s %d 0\n", dma ? "dma" : "registers", a <= kHeadColBlock ? head_tile_cols(a) : dma ? head_wide_columns(c, a) : 128);
    } else if (what == 's') {  // columns, rows: floats for a draft head, for a base head
      printf("room %zu %zu\n", head_part_floats(a, b, kDraftPartFloats), head_part_floats(a, b, kHeadPartFloats));
    } else {  // B H nodes kv_cap dh; f32, rows as two bf16 numbers; a context for just these sequences and heads
      const long long bh = (long long)a * b, units = bh > 256 ? bh : 256;
      if (!f && e == 128 && attn_keys_by_wavefront(bh, c, d)) printf("few 1 1\n");
      else if (!f && e == 128) s = plan_bf16_128(a, b, c, d, units, g != 0);
      else s = plan_any(a, b, c, d, e, f != 0, 2 * units, g != 0);
      if (s.S) printf("%s %d %d\n", f || e != 128 ? "any" : attn_rows64(s, c) ? "rows64" : "rows128", s.QB, s.S);
    }
  }
}
"""


@functools.lru_cache(maxsize=None)
def _program():
    at = tempfile.mkdtemp(prefix="launch_plans")
    with open(os.path.join(at, "plan.cpp"), "w") as f:
        f.write(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, os.path.join(at, "plan.cpp"), "-o", os.path.join(at, "plan")], check=True)
    return os.path.join(at, "plan")


def ask(lines):
    """One (what, number, number) per line; a line is the rule's letter and its arguments."""
    text = "\n".join(" ".join(map(str, list(l) + [0] * (8 - len(l)))) for l in lines)
    out = subprocess.run([_program()], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
    return [(w, int(x), int(y)) for w, x, y in (l.split() for l in out if l)]


def draft_head(cols, D, Vp1, dtype, k):
    """('ranges', tile columns, ranges), ('stream', column tiles, stages) or ('tile', tile columns, 0)."""
    return ask([("d", cols, D, Vp1, int("32" in str(dtype)), k)])[0]


def base_head(cols, D, V, dtype):
    """('ranges', tile columns, ranges) or ('tile', tile columns, rows)."""
    return ask([("b", cols, D, V, int("32" in str(dtype)))])[0]


def head_loop(cols, D, V, dtype, ranges=1):
    """('dma' or 'registers', columns of the base head's own tiles, 0): the tile loop that a head's tiles take."""
    return ask([("l", cols, D, V, int("32" in str(dtype)), ranges)])[0]


def head_room(cols, rows):
    """('room', floats for a draft head, for a base head): what a context of these limits keeps for partial sums."""
    return ask([("s", cols, rows)])[0]


def attention(B, H, nodes, kv_cap, dh, dtype, two_bf16=False):
    """(kernel, query blocks, key splits) in a context for B sequences and H heads."""
    return ask([("a", B, H, nodes, kv_cap, dh, int("32" in str(dtype)), int(two_bf16))])[0]
