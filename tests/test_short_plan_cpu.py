"""The kernel for few query rows, without a GPU: which problems it takes (the rule is plain C++, compiled here with the host
compiler), on both sides of its lines, and its registers and LDS."""
import os
import subprocess

import pytest

import paper_2312_11918_amd as fa2
from paper_2312_11918_amd import build
from test_gpu_short import CASES

PROGRAM = r"""
#include <stdio.h>
#include "fa2_short_plan.h"
int main() {
  int B, H, Nq, Nk, d, causal, sliced;
  while (scanf("%d %d %d %d %d %d %d", &B, &H, &Nq, &Nk, &d, &causal, &sliced) == 7)
    printf("%d\n", fa2::short_waves(B, H, Nq, Nk, d, causal != 0, sliced != 0));
}
"""


@pytest.fixture(scope="module")
def waves(tmp_path_factory):
    folder = tmp_path_factory.mktemp("short")
    source, program = folder / "short.cc", folder / "short"
    source.write_text(PROGRAM)
    csrc = os.path.dirname(build.SOURCES[0])
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", csrc, str(source), "-o", str(program)], check=True)

    def run(problems):
        text = "".join(" ".join(str(int(x)) for x in p) + "\n" for p in problems)
        out = subprocess.run([str(program)], input=text, stdout=subprocess.PIPE, text=True, check=True).stdout
        return [int(x) for x in out.split()]
    return run


# B, H, Nq, Nk, d, causal, slices to be had: wavefronts.  Measured on both sides of each line, see fa2_short_plan.h.
LINES = [
    ((1, 16, 512, 512, 128, 0, 0), 4), ((1, 17, 512, 512, 128, 0, 0), 0),        # a tile per CU
    ((1, 16, 768, 768, 128, 0, 0), 4), ((1, 17, 768, 768, 128, 0, 0), 0),
    ((1, 32, 512, 512, 64, 0, 0), 4), ((1, 32, 768, 768, 64, 0, 0), 0), ((1, 64, 256, 256, 64, 0, 0), 0),
    ((1, 16, 1111, 1111, 128, 1, 0), 4), ((1, 16, 1536, 1536, 128, 1, 0), 0),
    ((1, 128, 205, 205, 128, 1, 0), 4), ((1, 128, 256, 256, 128, 1, 0), 0), ((1, 128, 128, 128, 128, 1, 0), 0),
    ((1, 128, 256, 256, 256, 1, 0), 2), ((1, 128, 128, 128, 256, 1, 0), 2), ((1, 200, 128, 128, 256, 1, 0), 0),
    ((1, 4, 1000, 1000, 256, 0, 0), 4), ((1, 1, 999, 1000, 256, 0, 0), 0),
    ((1, 8, 288, 288, 256, 0, 0), 4), ((1, 8, 256, 256, 256, 0, 0), 0), ((1, 8, 255, 256, 256, 0, 0), 4),   # the tile kernel's bits
    ((1, 1, 768, 768, 64, 0, 0), 4), ((1, 1, 769, 769, 64, 0, 0), 8),            # eight wavefronts
    ((1, 2, 64, 1399, 64, 0, 1), 8), ((1, 2, 64, 1400, 64, 0, 1), 0), ((1, 2, 64, 1400, 64, 0, 0), 8),   # slices
    ((1, 2, 64, 1024, 128, 0, 1), 0), ((1, 2, 1024, 1024, 128, 1, 1), 8),
    ((1, 1, 2, 2301, 64, 0, 0), 0),
    ((65535, 65535, 2147483647, 5, 64, 0, 0), 0),                                # no overflow
]


def test_lines_of_the_rule(waves):
    for (p, want), got in zip(LINES, waves([p for p, _ in LINES])):
        assert got == want, p


def test_the_gpu_cases_run_in_it(waves):
    problems = [(B, H, Nq, Nk, d, causal, 0) for B, H, Nq, Nk, d, _, causal, _, _ in CASES]
    for case, got in zip(CASES, waves(problems)):
        assert got == case[-1], case


def test_a_problem_that_it_takes_from_the_slices_asks_for_no_workspace(waves):
    problems = [(1, H, Nq, Nk, d, c, 1) for H in (1, 2, 7, 16) for Nq, Nk, c in ((64, 700, 0), (100, 1500, 0), (1300, 1300, 1), (2, 4096, 0))
                for d in (64, 128, 256)]
    for p, got in zip(problems, waves(problems)):
        need = fa2.fa2_workspace_bytes(*p[:5], fa2.FA2_MASK_CAUSAL if p[5] else fa2.FA2_MASK_NONE)
        assert got == 0 or need == 0, p


def test_kernels_fit_their_launches():
    kernels = build.resource_usage(build.SHORT_SOURCES)
    # 2 element types x (4 and 8 wavefronts at d = 64 and 128, 4 at d = 256, with and without the mask, 2 at d = 256 with it)
    assert len(kernels) == len({k["name"] for k in kernels}) == 2 * (2 * (2 * 2 + 1) + 1)
    for k in kernels:
        waves = int(k["name"].split(" wavefronts")[0].split()[-1])
        per_simd = {"64": 4, "128": 2, "256": 1}[k["name"].split("d=")[1].split(",")[0]]
        groups = per_simd * 4 // waves   # workgroups per CU
        assert k["scratch_bytes_per_lane"] == 0 and k["waves_per_simd"] >= per_simd, k
        assert groups * k["lds_bytes_per_workgroup"] <= 160 * 1024, k
