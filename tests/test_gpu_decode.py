"""GPU parity of the single-query kernel (Nq == 1) against the fp64 CPU oracle: key counts around its step sizes and its
splits, with the keys split (workspace) and unsplit (none).  P and O are held in fp32 until O is rounded once, so O may
be off by half an ulp of the 16-bit type (2^-11 / 2^-8 relative) plus fp32 sums: checked as |dO| <= |O| ulp/2 + 1e-5."""
import numpy as np
import pytest

import oracle
import paper_2312_11918_amd as fa2
from test_gpu_ragged import PAD, SENT16, SENT32, _guarded, _make
from _gpu_common import mask_by_lowest_value, torch_gpu

pytestmark = pytest.mark.gpu


def _decode(qb, kb, vb, dtype, scale, split):
    torch = torch_gpu()
    B, _, H, d = qb.shape
    Nk = kb.shape[1]
    q, k, v = (_guarded(x, dtype)[0] for x in (qb, kb, vb))
    o, o_whole = _guarded(np.full(qb.shape, SENT16, dtype=np.uint16), dtype)
    lse_whole = torch.full((B * H + 2 * PAD,), float(SENT32), dtype=torch.float32, device="cuda")
    lse = lse_whole[PAD:PAD + B * H].view(B, H, 1)
    if split:
        fa2.fa2_fwd(q, k, v, scale, out=o, lse=lse)
    else:
        rc = fa2.fa2_fwd_qk_raw(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), lse.data_ptr(), B, H, 1, Nk, d, scale,
                                fa2.FA2_FP16 if dtype == "fp16" else fa2.FA2_BF16, fa2.FA2_MASK_NONE,
                                torch.cuda.current_stream().cuda_stream)
        assert rc == fa2.FA2_OK
    torch.cuda.synchronize()
    ow, lw = o_whole.cpu().numpy().view(np.uint16), lse_whole.cpu().numpy()
    assert np.all(ow[:PAD] == SENT16) and np.all(ow[PAD + qb.size:] == SENT16), "O was written outside its bounds"
    assert np.all(lw[:PAD] == SENT32) and np.all(lw[PAD + B * H:] == SENT32), "LSE was written outside its bounds"
    return o.double().cpu().numpy(), lse.double().cpu().numpy()


@pytest.mark.parametrize("B,H,Nk,d,dtype,outliers", [
    (1, 1, 1, 64, "fp16", 0.0),          # one key: O = V_0
    (2, 3, 7, 256, "bf16", 0.0),         # d = 256: steps of 8 keys
    (2, 3, 9, 256, "fp16", 0.0),
    (1, 2, 16, 128, "bf16", 0.0),        # steps of 16
    (1, 2, 17, 128, "fp16", 0.0),
    (3, 1, 31, 64, "bf16", 0.0),         # steps of 32
    (3, 2, 33, 64, "fp16", 0.02),
    (2, 5, 128, 128, "bf16", 0.0),       # a full step of eight wavefronts
    (2, 5, 129, 128, "fp16", 0.0),       # one key past it
    (2, 5, 257, 128, "fp16", 0.0),       # one key past two
    (3, 2, 130, 64, "bf16", 0.0),        # eight wavefronts of which three hold no key
    (33, 8, 300, 64, "bf16", 0.0),       # more heads than CUs
    (70, 8, 513, 128, "fp16", 0.0),      # ... and than twice the CUs
    (1, 2, 2047, 64, "fp16", 0.0),       # the last length that is not split at d = 64
    (1, 2, 2048, 64, "bf16", 0.0),       # the first that is
    (1, 2, 1024, 128, "bf16", 0.0),      # the first at d = 128: a step of keys per wavefront
    (1, 1, 513, 256, "fp16", 0.01),
    (13, 10, 1100, 128, "fp16", 0.0),    # 130 heads: several rounds of workgroups
    (12, 24, 1024, 128, "bf16", 0.0),    # 288 heads, split as well
    (3, 7, 5001, 128, "fp16", 0.01),     # uneven splits
    (1, 32, 16001, 64, "fp16", 0.0),
    (2, 16, 32768, 128, "bf16", 0.0),
])
@pytest.mark.parametrize("split", [True, False])
def test_single_query_parity(B, H, Nk, d, dtype, outliers, split):
    print(f"decode B={B} H={H} Nk={Nk} d={d} {dtype} split={split}", flush=True)
    qb, kb, vb = _make(B, H, 1, Nk, d, dtype, 5000 + Nk + d, outliers)
    scale = float(np.float32(d) ** np.float32(-0.5))
    torch_gpu()   # torch first: libfa2 then finds the HIP runtime that torch has loaded
    assert (fa2.fa2_workspace_bytes(B, H, 1, Nk, d) > 0) == (Nk * d >= 128 * 1024 and B * H < 512)
    o_ref, lse_ref = oracle.attention(*(oracle.widen(x, dtype) for x in (qb, kb, vb)), scale)
    o, lse = _decode(qb, kb, vb, dtype, scale, split)
    half_ulp = 2.0 ** (-11 if dtype == "fp16" else -8)
    assert np.all(np.abs(o - o_ref) <= np.abs(o_ref) * half_ulp + 1e-5)
    assert np.all(np.abs(lse - lse_ref) <= 1e-5 * np.maximum(1.0, np.abs(lse_ref)))


@pytest.mark.parametrize("H,Nk,d,dtype", [(8, 32768, 256, "fp16"), (4, 65536, 128, "bf16"), (4, 131072, 64, "fp16")])
@pytest.mark.parametrize("split", [True, False])
def test_single_query_large_logits_over_many_steps(H, Nk, d, dtype, split):
    # A common part of 200 ... 400 in the scaled logits of a head, 512 steps of the unsplit kernel, V larger in the early
    # keys than in the late ones: an error of the running rescale grows with every step and shows in LSE and O.
    # LSE: a logit is a sum of fp32 products, 8 in a lane and log2(d / 8) exchanges, then scaled, its reference rounded
    # and log2 e rounded: at most 16 roundings of 2^-24 of the sum of their absolute values, i.e. 1e-6 of about |LSE|.
    # O: the same error enters the weights, common to all keys but for the part that N(0,1) varies: 1e-4 of the largest |V|.
    print(f"decode offsets Nk={Nk} d={d} {dtype} split={split}", flush=True)
    torch = torch_gpu()
    qb, kb, vb = _make(1, H, 1, Nk, d, dtype, 6100 + d, 0.0)
    tdt = torch.float16 if dtype == "fp16" else torch.bfloat16
    q, k, v = (torch.from_numpy(x.view(np.int16)).view(tdt).clone() for x in (qb, kb, vb))
    q[..., 0] = 16.0
    k[..., 0] = torch.linspace(200.0, 400.0, H) * (d ** 0.5 / 16.0)
    v[:, :Nk // 2] += 1.0
    qb, kb, vb = (x.view(torch.int16).numpy().view(np.uint16) for x in (q, k, v))
    scale = float(np.float32(d) ** np.float32(-0.5))
    o_ref, lse_ref = oracle.attention(*(oracle.widen(x, dtype) for x in (qb, kb, vb)), scale)
    o, lse = _decode(qb, kb, vb, dtype, scale, split)
    print(f"max|dLSE|/LSE {np.max(np.abs(lse - lse_ref) / lse_ref):.2e} max|dO| {np.abs(o - o_ref).max():.2e}", flush=True)
    assert np.all(np.abs(lse - lse_ref) <= 1e-6 * lse_ref)
    half_ulp = 2.0 ** (-11 if dtype == "fp16" else -8)
    assert np.all(np.abs(o - o_ref) <= np.abs(o_ref) * half_ulp + 1e-4 * np.abs(oracle.widen(vb, dtype)).max())


@pytest.mark.parametrize("Nk,live,d,dtype", [
    (600, 30, 128, "bf16"),      # lane groups and wavefronts with masked keys only
    (4096, 1000, 128, "bf16"),   # splits with masked keys only
    (9000, 1, 64, "bf16"),
    (3000, 700, 256, "bf16"),
    (4096, 1000, 128, "fp16"),   # -65504: no overflow
])
@pytest.mark.parametrize("split", [True, False])
def test_single_query_keys_masked_by_the_lowest_value(Nk, live, d, dtype, split):
    # the scaled logits of masked keys overflow fp32 in bf16 (lowest value * log2 e); finite inputs, so O and LSE are those of
    # the live keys
    print(f"decode masked keys Nk={Nk} live={live} d={d} {dtype} split={split}", flush=True)
    qb, kb, vb = _make(1, 3, 1, Nk, d, dtype, 7100 + Nk + d, 0.0)
    qb, kb = mask_by_lowest_value(qb, kb, live, dtype)
    o_ref, lse_ref = oracle.attention(oracle.widen(qb, dtype), oracle.widen(kb[:, :live].copy(), dtype),
                                      oracle.widen(vb[:, :live].copy(), dtype), 1.0)
    o, lse = _decode(qb, kb, vb, dtype, 1.0, split)
    half_ulp = 2.0 ** (-11 if dtype == "fp16" else -8)
    assert np.all(np.abs(o - o_ref) <= np.abs(o_ref) * half_ulp + 1e-5)
    assert np.all(np.abs(lse - lse_ref) <= 1e-5 * np.maximum(1.0, np.abs(lse_ref)))


@pytest.mark.parametrize("Nk,d,dtype", [
    (4096, 64, "fp16"),     # 16 splits of a step per wavefront: the last count merged by one thread per column
    (4352, 64, "bf16"),     # 17: the first merged by lane groups
    (8192, 128, "bf16"),    # 64: every lane group holds four
    (8320, 128, "fp16"),    # 65: one of them a fifth
    (16384, 256, "bf16"),   # 256, the most of one head: four rounds of four
])
def test_single_query_merge_of_many_splits(Nk, d, dtype):
    print(f"decode merge Nk={Nk} d={d} {dtype}", flush=True)
    torch_gpu()
    splits = fa2.fa2_workspace_bytes(1, 1, 1, Nk, d) // (4 * (d + 2))
    assert splits == Nk * d // (8 * 4 * 512)
    qb, kb, vb = _make(1, 1, 1, Nk, d, dtype, 8100 + Nk + d, 0.02)
    scale = float(np.float32(d) ** np.float32(-0.5))
    o_ref, lse_ref = oracle.attention(*(oracle.widen(x, dtype) for x in (qb, kb, vb)), scale)
    o, lse = _decode(qb, kb, vb, dtype, scale, True)
    half_ulp = 2.0 ** (-11 if dtype == "fp16" else -8)
    assert np.all(np.abs(o - o_ref) <= np.abs(o_ref) * half_ulp + 1e-5)
    assert np.all(np.abs(lse - lse_ref) <= 1e-5 * np.maximum(1.0, np.abs(lse_ref)))
