"""Which problems run with the softmax mixed into the MFMAs, of those that are not of few query rows (test_routes_cpu.py), and the
compiled form of that kernel, on the CPU."""
import os
import subprocess

import pytest

from paper_2312_11918_amd import build
from test_gpu_stage import CASES, CASES_256, COMPANY, SAME_BITS, SINKING

PROGRAM = r"""
#include <stdio.h>
#include "fa2_stage_plan.h"
int main() {
  int B, H, Nq, Nk, d, causal;
  while (scanf("%d %d %d %d %d %d", &B, &H, &Nq, &Nk, &d, &causal) == 6)
    printf("%d\n", fa2::stage_accepts(B, H, Nq, Nk, d, causal != 0) && !fa2::split_plan(B, H, Nq, Nk, d, causal != 0, true).use);
}
"""


@pytest.fixture(scope="module")
def taken(tmp_path_factory):
    folder = tmp_path_factory.mktemp("plan")
    source, program = folder / "plan.cc", folder / "plan"
    source.write_text(PROGRAM)
    csrc = os.path.dirname(build.SOURCES[0])
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", csrc, str(source), "-o", str(program)], check=True)

    def run(problems):
        text = "".join(" ".join(str(int(x)) for x in p) + "\n" for p in problems)
        out = subprocess.run([str(program)], input=text, stdout=subprocess.PIPE, text=True, check=True).stdout
        return [line == "1" for line in out.split()]
    return run


def test_the_parity_cases_are_taken(taken):
    assert all(taken([(B, H, Nq, Nk, 256, causal) for B, H, Nq, Nk, _, causal, _ in CASES_256]))
    assert all(taken([(B, H, Nq, Nk, 64, causal) for B, H, Nq, Nk, _, causal, _ in CASES] + [(26, 16, 256, n, 64, 0) for n in (128, 256)]))
    assert all(taken([(B, H, Nq, Nk, d, causal) for B, H, Nq, Nk, d, _, causal in SINKING]))
    assert all(taken([(*sizes, d, 0) for d, sizes in COMPANY.items()] + [(B, H, N, N, d, 0) for B, H, N, d, _ in SAME_BITS]))


# measured with both launches, one clearly ahead
AHEAD = [(1, 32, 16384, 0), (32, 16, 512, 0), (2, 6, 9984, 0), (4, 16, 2816, 0), (64, 24, 130, 0), (10, 8, 1265, 0), (1, 32, 16384, 1),
         (5, 8, 6656, 1), (2, 12, 5555, 1), (4, 32, 4096, 1)]
BEHIND = [(6, 2, 6247, 0), (4, 6, 6016, 0), (13, 32, 384, 0), (26, 6, 1664, 0), (63, 6, 83, 0), (23, 8, 512, 0), (1, 8, 13184, 1),
          (12, 32, 476, 1), (29, 24, 640, 1), (1, 2, 256, 0), (1, 8, 3000, 0),
          (22, 32, 256, 0), (64, 16, 256, 0), (78, 12, 512, 0), (43, 12, 706, 0), (56, 8, 896, 0),   # short: starts and ends count
          (1, 16, 8036, 1), (2, 16, 4096, 1), (1, 32, 3912, 1), (3, 16, 3968, 1), (2, 32, 2944, 1)]   # pairs of whole rounds
# B, H, Nq, Nk
AHEAD_QK = [(22, 8, 3527, 167), (63, 8, 650, 190), (26, 16, 256, 119)]
BEHIND_QK = [(21, 32, 256, 71), (27, 12, 450, 117), (44, 8, 512, 72), (26, 24, 782, 127), (98, 2, 2644, 384)]

AHEAD_256 = [(4, 8, 4095, 0), (6, 12, 1000, 0), (11, 8, 777, 0), (2, 16, 1024, 0), (27, 6, 768, 0), (2, 6, 2048, 0), (9, 8, 2709, 1),
             (2, 24, 3633, 1), (8, 8, 2816, 1)]
BEHIND_256 = [(32, 16, 512, 0), (16, 16, 1024, 0), (4, 8, 4096, 0), (17, 24, 74, 0), (8, 16, 2048, 1), (32, 16, 512, 1), (7, 32, 768, 1),
              (1, 16, 4096, 1), (3, 6, 3328, 1)]


def test_the_rule_follows_the_measurements(taken):
    got = taken([(B, H, N, N, 64, causal) for B, H, N, causal in AHEAD + BEHIND])
    assert got == [True] * len(AHEAD) + [False] * len(BEHIND)
    got = taken([(B, H, Nq, Nk, 64, 0) for B, H, Nq, Nk in AHEAD_QK + BEHIND_QK])
    assert got == [True] * len(AHEAD_QK) + [False] * len(BEHIND_QK)
    assert not any(taken([(32, 16, 512, 512, d, 0) for d in (128, 256)]))
    got = taken([(B, H, N, N, 256, causal) for B, H, N, causal in AHEAD_256 + BEHIND_256])
    assert got == [True] * len(AHEAD_256) + [False] * len(BEHIND_256)


def test_the_kernels_fit_their_registers_without_scratch():
    kernels = build.resource_usage(build.STAGE_SOURCES)
    assert len({k["name"] for k in kernels}) == 2 * 2 * 4   # element types, head dimensions, causal mask, partial tiles
    for k in kernels:
        per_simd = 2 if "d=64" in k["name"] else 1   # wavefronts; as many workgroups per CU
        assert per_simd * (k["vgprs"] + k["agprs"]) <= 512 and k["waves_per_simd"] >= per_simd, k
        assert k["scratch_bytes_per_lane"] == 0 and per_simd * k["lds_bytes_per_workgroup"] <= 160 * 1024, k
