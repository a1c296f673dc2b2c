"""GPU parity of the kernel with the softmax mixed into the MFMAs (d = 64 with many Q tiles, d = 256) against the fp64 CPU
oracle on guarded buffers, with the tolerances of the other launches, and against the tile kernel bit by bit, at
the edges of its stages (32 keys), tiles (64 keys) and workgroups (256 or 128 rows)."""
import numpy as np
import pytest

import oracle
import paper_2312_11918_amd as fa2
from test_gpu_ragged import _check, _make, _run
from _gpu_common import mask_by_lowest_value, run_gpu

pytestmark = pytest.mark.gpu

# B, H, Nq, Nk, dtype, causal, outliers: all of them problems that stage_accepts() takes (test_stage_plan_cpu.py).  Outlier keys
# make P nearly one-hot and outputs as large as V: in bf16 half an ulp of an output in [4, 8) is 1.6e-2, beyond the tolerance of
# 1e-2 before any arithmetic (2.1e-2 seen at 65 keys with outliers), so they go with fp16 (half an ulp there 2e-3).
CASES = [
    (26, 16, 256, 1, "fp16", False, 0.0),        # one key: one stage with one column
    (26, 16, 255, 32, "bf16", False, 0.0),       # one stage, the other half of the tile masked
    (26, 16, 193, 33, "fp16", False, 0.0),       # two stages; a last wavefront of one row
    (26, 16, 192, 64, "fp16", False, 0.0),       # a wavefront without a row
    (26, 16, 250, 65, "fp16", False, 0.02),      # a second tile of one key
    (32, 16, 256, 128, "fp16", False, 0.0),      # whole tiles, no boundary with a refill
    (13, 16, 512, 192, "bf16", False, 0.0),
    (26, 16, 256, 448, "fp16", False, 0.05),     # odd count of tiles; the reference point moves
    (8, 25, 511, 257, "fp16", False, 0.0),
    (8, 9, 2048, 2048, "bf16", True, 0.0),       # whole tiles; heads in groups
    (7, 9, 2049, 2049, "fp16", True, 0.01),      # heads not a multiple of 8; a last Q tile of one row
    (8, 9, 1985, 1985, "fp16", True, 0.0),
]
# (those of few tiles run with 32 query rows per workgroup, see test_routes_cpu.py; the same edges with more heads are in
# test_gpu_launches.py)
CASES_256 = [
    (2, 3, 130, 129, "fp16", False, 0.0),        # an odd count of stages and tiles, a last tile of one key
    (2, 3, 128, 160, "bf16", False, 0.0),        # the last tile half masked
    (3, 2, 33, 191, "fp16", False, 0.02),        # wavefronts without a row; the reference point moves
    (3, 5, 97, 193, "bf16", False, 0.0),         # four tiles, the last of one key
    (2, 3, 256, 256, "fp16", False, 0.05),       # whole tiles
    (2, 3, 2, 255, "fp16", False, 0.0),
    (4, 21, 1537, 1537, "fp16", True, 0.01),     # odd counts of Q tiles, the last of one row; heads not a multiple of 8
    (8, 8, 2176, 2176, "bf16", True, 0.0),       # whole tiles, heads in groups
]


@pytest.mark.parametrize("d,B,H,Nq,Nk,dtype,causal,outliers", [(64, *c) for c in CASES] + [(256, *c) for c in CASES_256])
def test_stage_parity(d, B, H, Nq, Nk, dtype, causal, outliers):
    print(f"stage case d={d} B={B} H={H} Nq={Nq} Nk={Nk} {dtype} causal={causal}", flush=True)
    qb, kb, vb = _make(B, H, Nq, Nk, d, dtype, 47000 + Nq + Nk, outliers)
    scale = d ** -0.5
    o_ref, lse_ref = oracle.attention(*(oracle.widen(x, dtype) for x in (qb, kb, vb)), scale, causal=causal)
    o, lse = _run(qb, kb, vb, dtype, scale, causal)
    _check(o, lse, o_ref, lse_ref, "stage")


COMPANY = {64: (26, 16, 256, 200), 256: (9, 16, 130, 200)}   # B, H, Nq, Nk of staged problems


@pytest.mark.parametrize("d,live", [(d, n) for d in (64, 256) for n in (1, 33, 64, 100)])
def test_keys_masked_by_the_lowest_value(d, live):
    # scaled logits of masked keys overflow fp32; O and LSE are those of the live keys, also over stages that hold none
    print(f"stage masked keys d={d} live={live}", flush=True)
    B, H, Nq, Nk = COMPANY[d]
    qb, kb, vb = _make(B, H, Nq, Nk, d, "bf16", 9300 + live)
    qb, kb = mask_by_lowest_value(qb, kb, live, "bf16")
    o_ref, lse_ref = oracle.attention(oracle.widen(qb, "bf16"), oracle.widen(kb[:, :live].copy(), "bf16"),
                                      oracle.widen(vb[:, :live].copy(), "bf16"), 1.0)
    o, lse = _run(qb, kb, vb, "bf16", 1.0)
    _check(o, lse, o_ref, lse_ref, "masked keys")


@pytest.mark.parametrize("d,dead", [(64, 40), (256, 70)])
def test_first_keys_masked_by_the_lowest_value(d, dead):
    # the first stage (d = 256: the first tile) holds no live key: the reference is or stops at the lowest finite number, then moves
    B, H, Nq, Nk = COMPANY[d]
    print(f"stage first keys masked d={d}", flush=True)
    qb, kb, vb = _make(B, H, Nq, Nk, d, "bf16", 9400)
    qb, kb = mask_by_lowest_value(qb, kb[:, ::-1].copy(), Nk - dead, "bf16")
    kb, live = kb[:, ::-1].copy(), slice(dead, None)   # masked keys first
    o_ref, lse_ref = oracle.attention(oracle.widen(qb, "bf16"), oracle.widen(kb[:, live].copy(), "bf16"),
                                      oracle.widen(vb[:, live].copy(), "bf16"), 1.0)
    o, lse = _run(qb, kb, vb, "bf16", 1.0)
    _check(o, lse, o_ref, lse_ref, "first keys masked")


@pytest.mark.parametrize("d,B,H,N", [(64, 26, 16, 256), (256, 2, 3, 256)])
def test_a_rows_bits_do_not_depend_on_its_neighbours(d, B, H, N):
    # which rows move their reference is decided from their own values: outlier keys, and the same rows in other company
    print(f"stage bits d={d}", flush=True)
    qb, kb, vb = _make(B, H, N, N, d, "fp16", 47777, 0.05)
    o, lse = _run(qb, kb, vb, "fp16", d ** -0.5)
    order = np.random.Generator(np.random.PCG64(3)).permutation(N)
    o2, lse2 = _run(qb[:, order].copy(), kb, vb, "fp16", d ** -0.5)
    assert np.array_equal(o[:, order], o2) and np.array_equal(lse[:, :, order], lse2)


# B, H, N, d, dtype: square, staged (test_stage_plan_cpu.py), whole and partial tiles
SAME_BITS = [
    (26, 16, 256, 64, "fp16"),
    (26, 16, 233, 64, "bf16"),
    (8, 25, 511, 64, "fp16"),
    (2, 3, 256, 256, "bf16"),
    (2, 3, 257, 256, "fp16"),
    (2, 3, 191, 256, "bf16"),
]


@pytest.mark.parametrize("B,H,N,d,dtype", SAME_BITS)
def test_the_tile_kernels_bits(B, H, N, d, dtype):
    # N(0,1) inputs, no row of which has a key 8 (log2) above the maximum of its first 64: no reference moves, and both kernels
    # sum in one order
    print(f"stage against tile kernel B={B} H={H} N={N} d={d} {dtype}", flush=True)
    bits = _make(B, H, N, N, d, dtype, 49000 + N + d)
    o, lse = run_gpu(*bits, dtype, d ** -0.5, bits=True)
    o2, lse2 = run_gpu(*bits, dtype, d ** -0.5, variant=fa2.FA2_VARIANT_NARROW, bits=True)
    assert np.array_equal(o, o2) and np.array_equal(lse, lse2)


# B, H, Nq, Nk, d, dtype, causal: 12 tiles and more of keys that drive the reference point (test_stage_plan_cpu.py: all staged).  bf16
# only where P = 1 and 2^8 and few heads keep |O| below 4, half an ulp of which is 7.8e-3.
SINKING = [
    (26, 16, 256, 768, 64, "fp16", False),
    (26, 16, 250, 801, 64, "fp16", False),
    (8, 9, 2048, 2048, 64, "fp16", True),
    (7, 9, 2049, 2049, 64, "fp16", True),
    (9, 16, 130, 769, 256, "bf16", False),
    (9, 16, 256, 768, 256, "fp16", False),
    (4, 21, 1537, 1537, 256, "fp16", True),
]


@pytest.mark.parametrize("B,H,Nq,Nk,d,dtype,causal", SINKING)
def test_the_reference_point_never_falls(B, H, Nq, Nk, d, dtype, causal):
    # Every tile after the first: one key 8 (log2) above a level that sinks by 15 a tile, in the first half, whose sum it brings
    # to the limit exactly; the second half's keys, 15 below, push it past.  A reference that followed the second half's maximum
    # would sink with them and O and its sums grow by 2^15 a tile, beyond fp32 after 9.
    print(f"sinking reference B={B} H={H} Nq={Nq} Nk={Nk} d={d} {dtype} causal={causal}", flush=True)
    qb, kb, vb = _make(B, H, Nq, Nk, d, dtype, 48000 + Nq + d)
    logits = np.full(Nk, -225.0)                     # integers that both types hold
    logits[:64] = 0.0
    for t in range(1, 12):
        level = -15.0 * (t - 1)
        logits[64 * t:64 * t + 32] = level - 60.0
        logits[64 * t + 3] = level + 8.0
        logits[64 * t + 32:64 * t + 64] = level - 15.0
    bits = (lambda x: np.float16(x).view(np.uint16)) if dtype == "fp16" else \
        (lambda x: (np.float32(x).view(np.uint32) >> 16).astype(np.uint16))
    qb[...], kb[..., 0] = 0, bits(logits)[None, :, None]
    qb[..., 0] = bits(1.0)
    scale = 0.6931472                                # scale * log2(e) is exactly 1 in fp32
    assert np.float32(scale) * np.float32(1.44269504088896340736) == 1.0
    o_ref, lse_ref = oracle.attention(*(oracle.widen(x, dtype) for x in (qb, kb, vb)), scale, causal=causal)
    o, lse = _run(qb, kb, vb, dtype, scale, causal)
    _check(o, lse, o_ref, lse_ref, "sinking reference")
