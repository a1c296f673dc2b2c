"""GPU parity of the 256-row shape on partial tiles against the fp64 CPU oracle, on guarded buffers, and bit by bit against the
128-row shape: sizes at the edges of its tiles (256 rows, 64 keys, four of them a round of its buffers)."""
import numpy as np
import pytest

import oracle
import paper_2312_11918_amd as fa2
from test_gpu_ragged import _check, _make, _run
from _gpu_common import run_gpu

pytestmark = pytest.mark.gpu

# B, H, Nq, Nk, dtype, causal; all of them problems that wide_accepts() takes (test_wide_plan_cpu.py)
CASES = [
    (16, 16, 511, 511, "fp16", False),      # one row and key short of a tile
    (16, 16, 385, 385, "bf16", False),      # a last tile with one row past its first half, and keys that end as early
    (16, 16, 500, 129, "fp16", False),      # one round of the buffers: a tile with one key, and one with none
    (16, 16, 512, 193, "bf16", False),      # whole Q tiles; the last K/V tile with one key
    (16, 16, 450, 705, "fp16", False),      # three rounds, the last tile with one key
    (8, 4, 1921, 960, "bf16", False),       # one round of the CUs: no chain
    (16, 32, 511, 511, "fp16", True),
    (32, 16, 385, 385, "fp16", True),
    (8, 8, 1921, 1921, "fp16", True),       # one round of pairs
    (16, 16, 897, 897, "fp16", True),       # two rounds of pairs
]


@pytest.mark.parametrize("B,H,Nq,Nk,dtype,causal", CASES)
def test_wide_parity(B, H, Nq, Nk, dtype, causal):
    print(f"wide case B={B} H={H} Nq={Nq} Nk={Nk} {dtype} causal={causal}", flush=True)
    qb, kb, vb = _make(B, H, Nq, Nk, 128, dtype, 61000 + Nq + Nk)
    scale = 128 ** -0.5
    o_ref, lse_ref = oracle.attention(*(oracle.widen(x, dtype) for x in (qb, kb, vb)), scale, causal=causal)
    o, lse = _run(qb, kb, vb, dtype, scale, causal)
    _check(o, lse, o_ref, lse_ref, "wide")
    if Nq == Nk and not causal:   # what an explicit tile shape runs: the same sums in the same order
        o, lse = run_gpu(qb, kb, vb, dtype, scale, bits=True)
        o2, lse2 = run_gpu(qb, kb, vb, dtype, scale, variant=fa2.FA2_VARIANT_NARROW, bits=True)
        assert np.array_equal(o, o2) and np.array_equal(lse, lse2)
