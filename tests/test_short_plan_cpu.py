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
  int B, H, Nq, Nk, d, causal, may_slice;
  while (scanf("%d %d %d %d %d %d %d", &B, &H, &Nq, &Nk, &d, &causal, &may_slice) == 7) {
    const fa2::ShortPlan p = fa2::short_plan(B, H, Nq, Nk, d, causal != 0, may_slice != 0);
    printf("%d %d %d %d\n", p.waves, p.slices, p.chunk, p.items);
  }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    folder = tmp_path_factory.mktemp("short")
    source, program = folder / "short.cc", folder / "short"
    source.write_text(PROGRAM)
    csrc = os.path.dirname(build.SOURCES[0])
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", csrc, str(source), "-o", str(program)], check=True)

    def run(problems):
        text = "".join(" ".join(str(int(x)) for x in p) + "\n" for p in problems)
        out = subprocess.run([str(program)], input=text, stdout=subprocess.PIPE, text=True, check=True).stdout
        return [tuple(int(x) for x in line.split()) for line in out.splitlines()]
    return run


# B, H, Nq, Nk, d, causal, workspace: wavefronts, slices.  Measured on both sides of each line, see fa2_short_plan.h.
LINES = [
    ((1, 16, 512, 512, 128, 0, 1), (4, 1)), ((1, 17, 512, 512, 128, 0, 1), (0, 1)),        # a tile per CU
    ((1, 16, 768, 768, 128, 0, 1), (4, 1)), ((1, 17, 768, 768, 128, 0, 1), (0, 1)),
    ((1, 32, 512, 512, 64, 0, 1), (4, 1)), ((1, 32, 768, 768, 64, 0, 1), (0, 1)), ((1, 64, 256, 256, 64, 0, 1), (0, 1)),
    ((1, 16, 1111, 1111, 128, 1, 1), (4, 1)), ((1, 16, 1536, 1536, 128, 1, 1), (0, 1)),
    ((1, 128, 205, 205, 128, 1, 1), (4, 1)), ((1, 128, 256, 256, 128, 1, 1), (0, 1)), ((1, 128, 128, 128, 128, 1, 1), (0, 1)),
    ((1, 4, 2688, 2688, 128, 1, 1), (8, 1)), ((1, 4, 3600, 3600, 128, 1, 1), (0, 1)),
    ((1, 128, 256, 256, 256, 1, 1), (2, 1)), ((1, 128, 128, 128, 256, 1, 1), (2, 1)), ((1, 200, 128, 128, 256, 1, 1), (0, 1)),
    ((1, 8, 288, 288, 256, 0, 1), (4, 1)), ((1, 8, 256, 256, 256, 0, 1), (0, 1)), ((1, 8, 255, 256, 256, 0, 1), (4, 1)),   # the tile kernel's bits
    ((1, 1, 768, 768, 64, 0, 1), (4, 1)), ((1, 1, 769, 769, 64, 0, 1), (8, 1)),            # eight wavefronts
    ((1, 36, 240, 1116, 128, 0, 1), (4, 1)), ((1, 40, 248, 1728, 128, 0, 1), (0, 1)),      # blocks in all
    ((1, 1, 128, 1430, 64, 0, 1), (4, 5)), ((1, 1, 128, 1430, 64, 0, 0), (8, 1)),          # slices, and the same problem without a workspace
    ((1, 2, 128, 896, 128, 0, 1), (8, 1)), ((1, 2, 128, 897, 128, 0, 1), (4, 3)),
    ((1, 16, 32, 3000, 128, 0, 1), (4, 11)), ((1, 16, 512, 8192, 128, 0, 1), (0, 1)), ((3, 16, 40, 8040, 64, 0, 1), (0, 1)),
    ((1, 6, 26, 1334, 256, 0, 1), (4, 5)), ((1, 2, 2688, 2688, 128, 1, 1), (8, 2)), ((1, 2, 1409, 1409, 256, 1, 1), (4, 4)),
    ((1, 1, 2, 2301, 64, 0, 0), (0, 1)),
    ((65535, 65535, 2147483647, 5, 64, 0, 1), (0, 1)), ((1, 1, 5, 2147483647, 64, 0, 1), (0, 1)),   # no overflow
]


def test_lines_of_the_rule(plan):
    for (p, want), got in zip(LINES, plan([p for p, _ in LINES])):
        assert got[:2] == want, (p, got)


def test_the_gpu_cases_run_in_it(plan):
    problems = [(B, H, Nq, Nk, d, causal, slices > 1) for B, H, Nq, Nk, d, _, causal, _, _, slices in CASES]
    for case, got in zip(CASES, plan(problems)):
        assert got[:2] == case[-2:], (case, got)


def test_slices_cover_the_keys_and_their_workspace(plan):
    problems = [(B, H, Nq, Nk, d, c, 1) for B, H in ((1, 1), (1, 7), (2, 16), (3, 16)) for d in (64, 128, 256)
                for Nq, Nk, c in ((64, 700, 0), (2, 4096, 0), (100, 1500, 0), (33, 9999, 0), (1300, 1300, 1), (2777, 2777, 1))]
    taken = 0
    for p, (waves, slices, chunk, items) in zip(problems, plan(problems)):
        B, H, Nq, Nk, d, causal, _ = p
        if waves == 0:
            continue
        n_q, n_b = (Nq + 31) // 32, (Nk + 31) // 32
        need = fa2.fa2_workspace_bytes(B, H, Nq, Nk, d, fa2.FA2_MASK_CAUSAL if causal else fa2.FA2_MASK_NONE)
        assert need == (B * H * n_q * slices * 32 * (d + 2) * 4 if slices > 1 else 0), p
        assert (slices - 1) * chunk < n_b <= slices * chunk, p   # every slice holds a key
        # under the mask slice s concerns the tiles from its first key on
        assert items == (sum(max(0, n_q - s * chunk) for s in range(slices)) if causal else slices * n_q), p
        assert slices == 1 or B * H * items <= 256, p
        taken += slices > 1
    assert taken > 20


def test_kernels_fit_their_launches():
    kernels = build.resource_usage(build.SHORT_SOURCES)
    # 2 element types x (4 and 8 wavefronts at d = 64 and 128, 4 at d = 256, with and without the mask, 2 at d = 256 with it)
    #                    and the merge of slices at every d, with and without the mask)
    assert len(kernels) == len({k["name"] for k in kernels}) == 2 * (2 * (2 * 2 + 1) + 1 + 2 * 3)
    for k in kernels:
        if "merge" in k["name"]:
            assert k["scratch_bytes_per_lane"] == 0 and k["waves_per_simd"] >= 7 and k["lds_bytes_per_workgroup"] == 0, k
            continue
        waves = int(k["name"].split(" wavefronts")[0].split()[-1])
        per_simd = {"64": 4, "128": 2, "256": 1}[k["name"].split("d=")[1].split(",")[0]]
        groups = per_simd * 4 // waves   # workgroups per CU
        assert k["scratch_bytes_per_lane"] == 0 and k["waves_per_simd"] >= per_simd, k
        assert groups * k["lds_bytes_per_workgroup"] <= 160 * 1024, k
