"""GPU parity of the kernel for few query rows against the fp64 CPU oracle, on guarded buffers, with the tolerances of the other
kernels: sizes around its tiles (32 rows), its blocks (32 keys) and a round of blocks over its wavefronts."""
import numpy as np
import pytest

import oracle
from test_gpu_ragged import _check, _make, _run
from _gpu_common import TOL_O_MAX, TOL_O_MEAN, mask_by_lowest_value, torch_gpu

pytestmark = pytest.mark.gpu

# B, H, Nq, Nk, d, dtype, causal, outliers, wavefronts, slices (with the workspace that the call takes)
CASES = [
    (1, 2, 2, 1, 64, "fp16", False, 0.0, 4, 1),          # one key: three wavefronts hold none
    (2, 3, 31, 31, 128, "bf16", False, 0.0, 4, 1),       # one short of a tile and of a block
    (1, 2, 32, 31, 256, "fp16", False, 0.0, 4, 1),
    (3, 1, 33, 33, 64, "bf16", False, 0.0, 4, 1),        # one past both
    (1, 5, 40, 127, 128, "fp16", False, 0.02, 4, 1),     # a round of blocks, its last one partial
    (1, 5, 64, 128, 256, "bf16", False, 0.0, 4, 1),      # a round
    (2, 3, 65, 129, 64, "fp16", False, 0.0, 4, 1),       # ... and one key of the next
    (2, 3, 5, 257, 128, "bf16", False, 0.0, 4, 1),       # ... of the one after
    (1, 7, 300, 290, 256, "fp16", False, 0.01, 4, 1),
    (1, 1, 700, 769, 64, "bf16", False, 0.0, 8, 1),      # eight wavefronts, the last round one block of one key
    (1, 40, 100, 1024, 128, "fp16", False, 0.02, 8, 1),   # whole rounds
    (1, 8, 33, 1025, 64, "fp16", False, 0.0, 8, 1),
    (1, 40, 130, 2300, 64, "bf16", False, 0.0, 8, 1),   # the most keys
    (2, 3, 2, 2, 64, "bf16", True, 0.0, 4, 1),           # causal
    (1, 2, 32, 32, 128, "fp16", True, 0.0, 4, 1),
    (2, 3, 33, 33, 256, "bf16", True, 0.0, 4, 1),        # a second tile of one row
    (1, 9, 129, 129, 64, "fp16", True, 0.02, 4, 1),      # a tile that starts a round
    (2, 8, 250, 250, 128, "bf16", True, 0.0, 4, 1),
    (1, 11, 161, 161, 128, "fp16", True, 0.0, 4, 1),     # heads that are no multiple of the XCDs
    (3, 20, 160, 160, 256, "bf16", True, 0.0, 2, 1),     # two wavefronts
    (1, 90, 95, 95, 256, "fp16", True, 0.0, 2, 1),
    (1, 100, 256, 256, 64, "fp16", True, 0.0, 4, 1),     # more tiles than fit the chip at once
    (1, 8, 1057, 1057, 64, "bf16", True, 0.01, 8, 1),
    (1, 5, 1300, 1300, 128, "fp16", True, 0.0, 8, 1),
    (1, 1, 128, 1430, 64, "fp16", False, 0.0, 4, 5),     # slices: nine blocks each, the last one of a partial block
    (1, 2, 2, 897, 128, "bf16", False, 0.0, 4, 3),       # ... ten, ten and nine, the last one of one key
    (1, 3, 33, 2048, 256, "fp16", False, 0.01, 4, 8),    # ... of two rounds each
    (1, 16, 65, 5001, 64, "bf16", False, 0.0, 8, 5),     # ... for eight wavefronts
    (1, 2, 32, 16384, 128, "fp16", False, 0.0, 4, 64),   # many
    (1, 2, 1281, 1281, 128, "bf16", True, 0.0, 4, 5),    # ... under the mask: the first tiles lie in one slice; a last tile of one row
    (1, 2, 2688, 2688, 128, "fp16", True, 0.01, 8, 2),
    (1, 1, 700, 700, 256, "fp16", True, 0.0, 4, 2),
]


@pytest.mark.parametrize("B,H,Nq,Nk,d,dtype,causal,outliers,waves,slices", CASES)
def test_short_parity(B, H, Nq, Nk, d, dtype, causal, outliers, waves, slices):
    print(f"short case B={B} H={H} Nq={Nq} Nk={Nk} d={d} {dtype} causal={causal}", flush=True)
    qb, kb, vb = _make(B, H, Nq, Nk, d, dtype, 52000 + Nq + Nk + d, outliers)
    scale = float(np.float32(d) ** np.float32(-0.5))
    o_ref, lse_ref = oracle.attention(*(oracle.widen(x, dtype) for x in (qb, kb, vb)), scale, causal=causal)
    first = o, lse = _run(qb, kb, vb, dtype, scale, causal)
    if dtype == "bf16":
        # P and O are rounded to bf16, each off by up to 2^-8 of its value, so an output beyond 2.56 / 2 (the first rows under the mask,
        # which have few keys to average) may be off by more than the 1e-2 of the other tests, by 2^-7 |O|.  The mean bound is
        # for all elements as they are.
        large = np.abs(o_ref) * 2.0 ** -7 > TOL_O_MAX
        eo = np.abs(o - o_ref)
        assert np.all(np.isfinite(o)) and np.all(eo[large] <= np.abs(o_ref)[large] * 2.0 ** -7), f"max |dO| {eo.max():.3e}"
        assert eo.mean() <= TOL_O_MEAN, f"mean |dO| {eo.mean():.3e}"
        o = np.where(large, o_ref, o)   # (what is left of the bound of 1e-2)
    _check(o, lse, o_ref, lse_ref, "short")
    o, lse = first
    again, lse_again = _run(qb, kb, vb, dtype, scale, causal)
    assert np.array_equal(o, again) and np.array_equal(lse, lse_again)   # summed in one order, whoever ends first


@pytest.mark.parametrize("Nq,Nk,live,d", [
    (64, 600, 30, 128),     # all wavefronts but the first hold masked keys only
    (20, 500, 129, 64),
    (40, 400, 1, 256),
    (2, 1200, 1000, 64),    # rounds of masked keys behind live ones
    (20, 3000, 100, 128),   # slices that hold none
    (2, 4000, 3000, 256),
])
def test_short_keys_masked_by_the_lowest_value(Nq, Nk, live, d):
    # scaled logits of masked keys overflow fp32 (lowest bf16 * log2 e); the inputs are finite, so O and LSE are those of the live
    # keys, also where a wavefront holds none
    print(f"short masked keys Nq={Nq} Nk={Nk} live={live} d={d}", flush=True)
    torch_gpu()
    qb, kb, vb = _make(1, 2, Nq, Nk, d, "bf16", 9300 + Nk + d)
    qb, kb = mask_by_lowest_value(qb, kb, live, "bf16")
    o_ref, lse_ref = oracle.attention(oracle.widen(qb, "bf16"), oracle.widen(kb[:, :live].copy(), "bf16"),
                                      oracle.widen(vb[:, :live].copy(), "bf16"), 1.0)
    o, lse = _run(qb, kb, vb, "bf16", 1.0)
    # one ulp of bf16 (P and O are rounded to it) of values up to max |V|
    assert np.all(np.isfinite(o)) and np.all(np.isfinite(lse))
    assert np.max(np.abs(o - o_ref)) <= 2.0 ** -7 * np.abs(oracle.widen(vb, "bf16")).max()
    assert np.max(np.abs(lse - lse_ref)) <= 1e-3
