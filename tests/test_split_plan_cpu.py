"""The choice between a whole launch and one with the keys cut, on the CPU: the plan is plain C++, compiled here with the host
compiler.  The cases are shapes that were measured with both launches, where one is clearly ahead."""
import os
import subprocess

import pytest

from paper_2312_11918_amd import build

PROGRAM = r"""
#include <stdio.h>
#include "fa2_split_plan.h"
int main() {
  int B, H, Nq, Nk, d, causal, may_slice;
  while (scanf("%d %d %d %d %d %d %d", &B, &H, &Nq, &Nk, &d, &causal, &may_slice) == 7) {
    const fa2::SplitPlan p = fa2::split_plan(B, H, Nq, Nk, d, causal != 0, may_slice != 0);
    printf("%d %d %d %d\n", p.use, p.chunk, p.slices, p.items);
  }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    folder = tmp_path_factory.mktemp("plan")
    source, program = folder / "plan.cc", folder / "plan"
    source.write_text(PROGRAM)
    csrc = os.path.dirname(build.SOURCES[0])
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", csrc, str(source), "-o", str(program)], check=True)

    def run(problems):
        text = "".join(" ".join(str(int(x)) for x in p) + "\n" for p in problems)
        out = subprocess.run([str(program)], input=text, stdout=subprocess.PIPE, text=True, check=True).stdout
        return [tuple(int(x) for x in line.split()) for line in out.splitlines()]
    return run


def test_d256_without_a_mask_is_never_the_whole_launch_in_another_kernel(plan):
    # one slice at d = 256 cuts nothing: the same workgroups and tiles in the slower partial-tile kernel
    problems = [(B, H, Nq, Nk, 256, 0, may) for B in (1, 2, 3, 4, 8, 16) for H in (1, 6, 7, 8, 12, 16)
                for Nq in (128, 200, 512, 1000, 1024, 2048, 4096) for Nk in (300, 512, 1024, 2000, 4096, 8192) for may in (0, 1)]
    for p, (use, _, slices, _) in zip(problems, plan(problems)):
        assert not use or slices > 1, p
