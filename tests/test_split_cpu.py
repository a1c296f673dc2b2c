"""Host logic and compiled form of the kernels that split the keys (no GPU): registers, and the scratch memory asked for."""
import pytest

import paper_2312_11918_amd as fa2
from paper_2312_11918_amd import build


def test_no_split_kernel_uses_scratch_memory():
    kernels = build.resource_usage(build.SPLIT_SOURCES)
    assert kernels
    bad = [(k["name"], k["scratch_bytes_per_lane"]) for k in kernels if k["scratch_bytes_per_lane"] != 0]
    assert not bad, f"kernels that spill to scratch: {bad}"


@pytest.mark.parametrize("B,H,Nk,d,splits", [
    (1, 32, 16001, 64, 8),      # 32 heads: one round of 256 workgroups
    (3, 12, 30000, 64, 7),      # 36 heads: 252
    (1, 1, 513, 256, 8),        # no more than a step of keys per wavefront
    (12, 24, 1500, 128, 4),     # 288 heads, 1.1 rounds: 4.5 rounds
    (16, 16, 2048, 128, 1),     # the heads fill the CUs
    (1, 32, 1023, 128, 1),      # too few keys
])
def test_decode_splits(B, H, Nk, d, splits):
    want = 0 if splits == 1 else B * H * splits * (d + 2) * 4   # O, maximum and sum in fp32 per split
    assert fa2.fa2_workspace_bytes(B, H, 1, Nk, d) == want


def test_workspace_of_refused_problems_is_zero():
    assert fa2.fa2_workspace_bytes(1, 1, 1, 4096, 96) == 0
    assert fa2.fa2_workspace_bytes(0, 1, 1, 4096, 64) == 0
    assert fa2.fa2_workspace_bytes(1, 1, 1, 4096, 64, fa2.FA2_MASK_CAUSAL) == 0
    assert fa2.fa2_fwd_ws_raw(4096, 4096, 4096, 4096, None, 1, 1, 1, 4096, 64, 0.125, 0, 0, 4104, 1 << 20) == fa2.FA2_ERR_INVALID_ARG


@pytest.mark.parametrize("B,H,Nq,Nk,d", [
    (1, 1, 1, 1 << 25, 64),              # a batch entry of K of 2^32 bytes
    (1, 1, 2, 1 << 25, 64),
    (1, 3, 128, 1 << 24, 128),
    (1, 1, (1 << 31) - 1, 600, 64),      # 2^31 - 1 queries: the count of Q tiles would overflow
    (1, 1, 600, (1 << 31) - 1, 64),
    (512, 1, 1, 1 << 22, 64),            # B * Nk past 2^31 - 1
])
def test_workspace_of_problems_past_the_size_limits_is_zero(B, H, Nq, Nk, d):
    assert fa2.fa2_fwd_ws_raw(4096, 4096, 4096, 4096, None, B, H, Nq, Nk, d, 0.125, 0, 0, None, 0) == fa2.FA2_ERR_UNSUPPORTED
    assert fa2.fa2_workspace_bytes(B, H, Nq, Nk, d) == 0


@pytest.mark.parametrize("mask", [-1, 2])
def test_workspace_of_an_unknown_mask_is_zero(mask):
    assert fa2.fa2_workspace_bytes(1, 1, 1, 4096, 64, mask) == 0


@pytest.fixture(scope="module")
def kernels():
    return build.resource_usage(build.SPLIT_SOURCES)


def test_every_split_kernel_is_reported(kernels):
    # 2 element types x 3 head dimensions x (the single-query kernel with and without split keys, its merge, the tile kernel
    #                                        with the keys cut and its merge, with and without the causal mask)
    names = {k["name"] for k in kernels}
    assert len(kernels) == len(names) == 2 * 3 * (2 + 1 + 2 + 2), sorted(names)


def test_split_kernels_fit_their_launches(kernels):
    for k in kernels:
        lds = k["lds_bytes_per_workgroup"]
        if "8 wavefronts" in k["name"]:      # halves: two wavefronts per SIMD, one workgroup per CU
            assert k["vgprs"] + k["agprs"] <= 256 and k["waves_per_simd"] >= 2 and lds <= 160 * 1024, k
        elif "fwd_kernel" in k["name"]:      # d = 256: one wavefront per SIMD
            assert k["vgprs"] + k["agprs"] <= 512 and lds <= 160 * 1024, k
        elif "decode_kernel" in k["name"]:   # latency is hidden by wavefronts: two workgroups of eight per CU
            assert k["waves_per_simd"] >= 4 and 2 * lds <= 160 * 1024, k
        else:
            assert k["waves_per_simd"] >= 7 and lds == 0, k
