"""Which kernel a call of the library runs in: the rules of the dispatch are plain C++ headers, compiled here with the host compiler
and asked in the order in which the library asks them."""
import functools
import os
import subprocess
import tempfile

import paper_2312_11918_amd as fa2
from paper_2312_11918_amd import build

PROGRAM = r"""
#include <stdio.h>
#include "fa2_short_plan.h"
#include "fa2_stage_plan.h"
#include "fa2_wide_plan.h"
static const char* route(int B, int H, int Nq, int Nk, int d, bool causal, bool workspace) {
  if (Nq == 1) return "decode";
  fa2::ShortPlan s = fa2::short_plan(B, H, Nq, Nk, d, causal, workspace);
  if (s.waves != 0) return s.slices > 1 ? "short slices" : "short";
  const fa2::SplitPlan p = fa2::split_plan(B, H, Nq, Nk, d, causal, workspace);
  if (p.use) return p.slices > 1 ? "slices" : d <= 128 ? "halves" : "single";
  if (fa2::stage_accepts(B, H, Nq, Nk, d, causal)) return "stage";
  if (fa2::wide_accepts(B, H, Nq, Nk, d, causal)) return "wide";
  return Nq % 128 == 0 && Nk % 128 == 0 ? "tiles" : "partial tiles";
}
int main() {
  int B, H, Nq, Nk, d, causal, workspace;
  while (scanf("%d %d %d %d %d %d %d", &B, &H, &Nq, &Nk, &d, &causal, &workspace) == 7)
    puts(route(B, H, Nq, Nk, d, causal != 0, workspace != 0));
}
"""


@functools.lru_cache(None)
def _program():
    folder = tempfile.mkdtemp()
    source, program = os.path.join(folder, "routes.cc"), os.path.join(folder, "routes")
    with open(source, "w") as f:
        f.write(PROGRAM)
    csrc = os.path.dirname(build.SOURCES[0])
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", csrc, source, "-o", program], check=True)
    return program


def routes(problems):
    """Of (B, H, Nq, Nk, d, causal, with the workspace that the call asks for): the names of their launches.  'tiles' are whole ones,
    in the 256-row shape where fa2_tile_shape() says so."""
    text = "".join(" ".join(str(int(x)) for x in p) + "\n" for p in problems)
    out = subprocess.run([_program()], input=text, stdout=subprocess.PIPE, text=True, check=True).stdout.splitlines()
    return [f"{r} of 256 rows" if r == "tiles" and fa2.fa2_tile_shape(*p[:5], fa2.FA2_MASK_CAUSAL if p[5] else fa2.FA2_MASK_NONE)
            == fa2.FA2_VARIANT_NARROW8 else r for r, p in zip(out, problems)]
