"""GPU parity of the launches that the dispatch leaves between those with test files of their own, against the fp64 CPU oracle on
guarded buffers with the tolerances of the others.  Which launch a problem gets is asserted on the CPU (test_routes_cpu.py), so that a
new rule of the dispatch cannot take these cases elsewhere unseen."""
import numpy as np
import pytest

import oracle
import paper_2312_11918_amd as fa2
from test_gpu_ragged import _check, _guarded, _make, _run
from _gpu_common import mask_by_lowest_value, torch_gpu

pytestmark = pytest.mark.gpu

# launch, B, H, Nq, Nk, d, dtype, causal, outliers.  Outlier keys make outputs as large as V, so they go with fp16.
CASES = [
    ("slices", 1, 8, 512, 8192, 64, "bf16", False, 0.0),          # slices of 128-row tiles and their merge
    ("slices", 1, 8, 500, 4097, 128, "bf16", False, 0.0),         # the last slice with one key in its last tile; dead wavefronts
    ("slices", 1, 2, 2304, 2304, 128, "fp16", False, 0.02),
    ("slices", 2, 8, 200, 4000, 256, "fp16", False, 0.01),        # d = 256 has no halves
    ("slices", 1, 3, 1408, 1408, 256, "bf16", False, 0.0),
    ("slices", 1, 2, 3700, 3700, 64, "fp16", True, 0.01),         # under the mask: the first Q tiles lie in one slice
    ("slices", 1, 2, 3713, 3713, 128, "bf16", True, 0.0),         # ... and a last one of one row
    ("slices", 1, 3, 1833, 1833, 256, "fp16", True, 0.0),
    ("slices", 2, 8, 801, 801, 256, "bf16", True, 0.0),
    ("halves", 5, 8, 512, 512, 64, "bf16", False, 0.0),
    ("halves", 8, 5, 500, 1100, 64, "fp16", False, 0.02),         # nine pairs of tiles, the last tile partial
    ("halves", 1, 24, 512, 512, 128, "bf16", False, 0.0),
    ("halves", 2, 10, 700, 1500, 128, "fp16", False, 0.01),
    ("halves", 3, 24, 385, 385, 64, "bf16", True, 0.0),
    ("halves", 3, 24, 257, 257, 128, "fp16", True, 0.0),
    ("single", 8, 5, 385, 385, 256, "bf16", True, 0.0),
    ("stage", 9, 16, 130, 129, 256, "fp16", False, 0.0),          # an odd count of stages and tiles, a last tile of one key
    ("stage", 9, 16, 128, 160, 256, "bf16", False, 0.0),          # the last tile half masked
    ("stage", 9, 16, 33, 191, 256, "fp16", False, 0.02),          # wavefronts without a row; the reference point moves
    ("stage", 18, 16, 97, 193, 256, "bf16", False, 0.0),          # four tiles, the last of one key
    ("stage", 18, 16, 2, 255, 256, "fp16", False, 0.0),
    ("partial tiles", 30, 12, 40, 77, 64, "bf16", False, 0.0),    # the 128-row shape as it is launched whole
    ("partial tiles", 30, 12, 129, 70, 128, "fp16", False, 0.02),
    ("partial tiles", 20, 24, 100, 100, 256, "bf16", False, 0.0),
    ("partial tiles", 50, 16, 330, 330, 64, "fp16", True, 0.0),   # pairs of Q tiles, the middle one unpaired
    ("partial tiles", 50, 16, 130, 130, 64, "bf16", True, 0.0),
    ("partial tiles", 16, 12, 700, 700, 128, "fp16", True, 0.01),   # the only kernel without row stores
    ("partial tiles", 50, 16, 129, 129, 128, "bf16", True, 0.0),
    ("partial tiles", 30, 16, 286, 286, 256, "fp16", True, 0.0),
    ("partial tiles", 30, 16, 130, 130, 256, "bf16", True, 0.0),
    ("tiles", 5, 16, 128, 128, 64, "bf16", False, 0.0),
    ("tiles", 3, 24, 128, 128, 128, "fp16", False, 0.0),
    ("tiles", 50, 16, 256, 256, 64, "bf16", True, 0.0),
    ("tiles", 16, 16, 384, 384, 128, "fp16", True, 0.02),
    ("tiles", 32, 12, 256, 256, 256, "bf16", True, 0.0),
    ("tiles of 256 rows", 16, 2, 2048, 2048, 64, "fp16", False, 0.01),
]


@pytest.mark.parametrize("launch,B,H,Nq,Nk,d,dtype,causal,outliers", CASES)
def test_launch_parity(launch, B, H, Nq, Nk, d, dtype, causal, outliers):
    print(f"{launch} case B={B} H={H} Nq={Nq} Nk={Nk} d={d} {dtype} causal={causal}", flush=True)
    torch_gpu()   # (torch's HIP runtime first, which the library then shares)
    mask = fa2.FA2_MASK_CAUSAL if causal else fa2.FA2_MASK_NONE
    assert (fa2.fa2_workspace_bytes(B, H, Nq, Nk, d, mask) > 0) == (launch == "slices")
    qb, kb, vb = _make(B, H, Nq, Nk, d, dtype, 71000 + Nq + Nk + d, outliers)
    scale = float(np.float32(d) ** np.float32(-0.5))
    o_ref, lse_ref = oracle.attention(*(oracle.widen(x, dtype) for x in (qb, kb, vb)), scale, causal=causal)
    o, lse = _run(qb, kb, vb, dtype, scale, causal)
    if dtype == "bf16":
        # P and O are rounded to 8 bits: beyond 2.56 / 2 (the first rows under the mask, which have few keys to average) the two
        # may be off by 2^-7 |O|, which is more than the 1e-2 of the others; the mean bound is for all elements as they are
        large = np.abs(o_ref) * 2.0 ** -7 > 1e-2
        assert np.all(np.isfinite(o)) and np.all(np.abs(o - o_ref)[large] <= np.abs(o_ref)[large] * 2.0 ** -7)
        assert np.mean(np.abs(o - o_ref)) <= 1e-3
        o = np.where(large, o_ref, o)
    _check(o, lse, o_ref, lse_ref, launch)


# launch with the workspace that the call takes and without one, B, H, Nq, Nk, live keys, d
MASKED = [
    ("slices", "halves", 1, 8, 512, 8192, 64, 64),        # half 1, and all slices but the first, see masked keys only
    ("slices", "halves", 1, 8, 512, 8192, 5000, 128),
    ("slices", "halves", 1, 8, 500, 4097, 1, 128),
    ("slices", "stage", 1, 2, 1500, 4000, 64, 256),       # slices without halves
    ("stage", "stage", 9, 16, 130, 200, 1, 256),
    ("stage", "stage", 9, 16, 130, 200, 100, 256),        # stages that hold masked keys only
    ("wide", "wide", 16, 16, 500, 129, 40, 128),
    ("wide", "wide", 16, 16, 450, 705, 300, 128),
    ("partial tiles", "partial tiles", 30, 12, 129, 300, 64, 128),
]


@pytest.mark.parametrize("with_ws,without,B,H,Nq,Nk,live,d", MASKED)
def test_keys_masked_by_the_lowest_value(with_ws, without, B, H, Nq, Nk, live, d):
    # scaled logits of masked keys overflow fp32 (lowest bf16 * log2 e); the inputs are finite, so O and LSE are those of the
    # live keys, also where a half, a slice or a stage holds none
    print(f"masked keys {with_ws} Nq={Nq} Nk={Nk} live={live} d={d}", flush=True)
    torch = torch_gpu()
    qb, kb, vb = _make(B, H, Nq, Nk, d, "bf16", 9500 + Nk + d)
    qb, kb = mask_by_lowest_value(qb, kb, live, "bf16")
    o_ref, lse_ref = oracle.attention(oracle.widen(qb, "bf16"), oracle.widen(kb[:, :live].copy(), "bf16"),
                                      oracle.widen(vb[:, :live].copy(), "bf16"), 1.0)
    results = [_run(qb, kb, vb, "bf16", 1.0)]
    if without != with_ws:
        q, k, v = (_guarded(x, "bf16")[0] for x in (qb, kb, vb))
        o = torch.full_like(q, float("nan"))
        lse = torch.full((B, H, Nq), float("nan"), dtype=torch.float32, device="cuda")
        assert fa2.fa2_fwd_qk_raw(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), lse.data_ptr(), B, H, Nq, Nk, d, 1.0,
                                  fa2.FA2_BF16, fa2.FA2_MASK_NONE, torch.cuda.current_stream().cuda_stream) == fa2.FA2_OK
        torch.cuda.synchronize()
        results.append((o.double().cpu().numpy(), lse.double().cpu().numpy()))
    for o, lse in results:
        # one ulp of bf16 (P and O are rounded to it) of values up to max |V|
        assert np.all(np.isfinite(o)) and np.all(np.isfinite(lse))
        assert np.max(np.abs(o - o_ref)) <= 2.0 ** -7 * np.abs(oracle.widen(vb, "bf16")).max()
        assert np.max(np.abs(lse - lse_ref)) <= 1e-3
