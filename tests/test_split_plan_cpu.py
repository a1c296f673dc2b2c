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


# B, H, N, d: causal problems, us whole / with single Q tiles in one slice (no workspace)
WHOLE = [
    (1, 16, 4096, 256), (1, 8, 4096, 256), (2, 8, 2048, 256),   # 144 / 160, 122 / 136, 69.6 / 72.2: whole tiles, chained
    (2, 12, 2560, 256), (3, 6, 3328, 256), (8, 2, 3840, 256),   # 96 / 104, 120 / 132, 135 / 145
    (10, 2, 3071, 256), (1, 16, 4059, 256), (99, 1, 462, 256),  # partial tiles: 117 / 122, 158 / 163, 36.1 / 38.4
    (8, 12, 512, 128), (7, 16, 384, 128), (5, 16, 640, 128),    # 19.3 / 20.9, 17.2 / 18.4, 21.4 / 22.1
    (8, 12, 512, 64), (7, 16, 384, 64),                         # 13.9 / 14.8, 12.6 / 13.2
]
SINGLE = [
    (1, 12, 3072, 128), (1, 24, 1536, 128), (8, 1, 4395, 128),  # 56.8 / 42.8, 33.8 / 25.4, 78.0 / 57.2
    (1, 32, 1127, 64), (2, 12, 1920, 64), (8, 2, 4736, 64),     # 21.0 / 15.4, 27.7 / 21.9, 80.8 / 66.9
    (16, 2, 2272, 256), (1, 24, 2632, 256), (3, 12, 1920, 256), # 176 / 123, 152 / 115, 139 / 100
    (8, 8, 512, 256), (2, 24, 731, 256),                        # 31.0 / 25.4, 40.4 / 33.5
]


def test_causal_problems_without_a_workspace(plan):
    problems = [(B, H, N, N, d, 1, 0) for B, H, N, d in WHOLE + SINGLE]
    for i, (p, (use, _, slices, _)) in enumerate(zip(problems, plan(problems))):
        assert slices == 1 and bool(use) == (i >= len(WHOLE)), p
