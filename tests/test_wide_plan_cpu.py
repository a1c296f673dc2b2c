"""Partial tiles in the 256-row shape, without a GPU: which problems run so (the rule is plain C++, compiled here with the host
compiler), on both sides of its lines, and the registers and LDS of its kernels."""
import os
import subprocess

from paper_2312_11918_amd import build
from test_gpu_wide import CASES

PROGRAM = r"""
#include <stdio.h>
#include "fa2_wide_plan.h"
int main() {
  int B, H, Nq, Nk, d, causal;
  while (scanf("%d %d %d %d %d %d", &B, &H, &Nq, &Nk, &d, &causal) == 6)
    printf("%d\n", fa2::wide_accepts(B, H, Nq, Nk, d, causal != 0));
}
"""

# B, H, Nq, Nk, d, causal; measured, see fa2_wide_plan.h
TAKEN = [(8, 16, 2047, 2047, 128, 0), (16, 16, 1000, 1000, 128, 0), (32, 16, 511, 511, 128, 0), (8, 16, 2047, 3000, 128, 0),
         (2, 16, 2000, 2000, 128, 0), (8, 16, 2047, 2047, 128, 1), (32, 16, 500, 500, 128, 1), (1, 16, 8100, 8100, 128, 1),
         (8, 16, 2048, 1000, 128, 0)]
LEFT = [(8, 16, 1900, 1900, 128, 0), (3, 16, 2000, 2000, 128, 0), (64, 16, 250, 250, 128, 0), (8, 16, 500, 5000, 128, 0),
        (8, 16, 2048, 2048, 128, 0), (8, 16, 2047, 2047, 64, 0), (8, 16, 1500, 1500, 128, 1), (16, 16, 700, 700, 128, 1),
        (65535, 65536, 2147483647, 5, 128, 0)]   # (and no overflow)


def test_lines_of_the_rule(tmp_path):
    source, program = tmp_path / "wide.cc", tmp_path / "wide"
    source.write_text(PROGRAM)
    csrc = os.path.dirname(build.SOURCES[0])
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", csrc, str(source), "-o", str(program)], check=True)
    problems = TAKEN + [(B, H, Nq, Nk, 128, causal) for B, H, Nq, Nk, _, causal in CASES] + LEFT
    text = "".join(" ".join(str(int(x)) for x in p) + "\n" for p in problems)
    out = subprocess.run([str(program)], input=text, stdout=subprocess.PIPE, text=True, check=True).stdout.split()
    for i, (p, got) in enumerate(zip(problems, out)):
        assert got == ("1" if i < len(problems) - len(LEFT) else "0"), p


STAGED = r"""
#include <stdio.h>
#include "fa2_wide_plan.h"
int main() {
  int j, Nk;
  while (scanf("%d %d", &j, &Nk) == 2) printf("%d\n", fa2::wide_staged_tile(j, Nk));
}
"""


def _in_range(lane_offset, scalar_offset, num_records):
    """The range check of a raw buffer load, in the unsigned 32-bit arithmetic that it is specified in."""
    return lane_offset < (num_records - scalar_offset) % 2 ** 32


def test_no_row_past_the_last_key_passes_the_range_check(tmp_path):
    source, program = tmp_path / "staged.cc", tmp_path / "staged"
    source.write_text(STAGED)
    csrc = os.path.dirname(build.SOURCES[0])
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", csrc, str(source), "-o", str(program)], check=True)
    # every count of keys that wide_accepts() takes, at both ends of the counts of tiles
    counts = [n for n in (*range(1, 1300), *range(8000, 8300)) if (n + 127) // 128 % 2 == 0]
    tiles = [(j, n) for n in counts for j in range((n + 255) // 256 * 4)]   # padded to whole rounds of the four buffers
    text = "".join(f"{j} {n}\n" for j, n in tiles)
    out = subprocess.run([str(program)], input=text, stdout=subprocess.PIPE, text=True, check=True).stdout.split()
    assert len(out) == len(tiles)
    wrapping = 0
    for (j, n), staged in zip(tiles, map(int, out)):
        assert staged == j or 64 * j >= n   # all tiles with a key as they are
        for heads in (1, 16):
            row_bytes = 256 * heads
            num_records = (n - 1) * row_bytes + 256
            for tile in {staged, j}:
                at = 64 * tile * row_bytes
                for row in {64 * tile + i for i in (0, 1, 31, 63)} | ({n - 1, n} & set(range(64 * tile, 64 * tile + 64))):
                    read = _in_range((row - 64 * tile) * row_bytes, at, num_records)
                    if tile == staged:
                        assert read == (row < n), (j, n, row)
                    wrapping += read and row >= n
    assert wrapping > 0   # what a load of a tile without keys would read


def test_kernels_fit_their_launches():
    kernels = build.resource_usage(build.WIDE_SOURCES)
    assert len(kernels) == 4   # 2 element types, with and without the causal mask
    for k in kernels:
        assert "d=128, 8 wavefronts" in k["name"] and "partial tiles" in k["name"], k
        assert k["scratch_bytes_per_lane"] == 0 and k["vgprs"] + k["agprs"] <= 256 and k["waves_per_simd"] >= 2, k
        assert k["lds_bytes_per_workgroup"] <= 160 * 1024, k
