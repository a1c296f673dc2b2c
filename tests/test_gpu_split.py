"""GPU parity of the launches that cut the keys (few Q tiles): over the wavefronts of a workgroup, over workgroups and their
merge, against the fp64 CPU oracle on guarded buffers, with the tolerances of the whole launches.  Which launch each case gets is in
test_routes_cpu.py; most of these get tiles of 32 rows, and test_gpu_launches.py has more of those that keep 128."""
import ctypes

import numpy as np
import pytest

import oracle
import paper_2312_11918_amd as fa2
from test_gpu_ragged import _check, _guarded, _make, _run
from _gpu_common import mask_by_lowest_value, torch_gpu

pytestmark = pytest.mark.gpu

# B, H, Nq, Nk, d, dtype, causal, outliers, sliced (over workgroups): sizes at the edges of tiles of 64 keys, pairs and fours of
# them, and of slices; Q tiles with dead wavefronts
CASES = [
    (1, 2, 129, 1500, 128, "fp16", False, 0.0, True),
    (1, 2, 128, 641, 128, "bf16", False, 0.0, False),     # a last tile of one key
    (2, 3, 100, 2000, 64, "fp16", False, 0.02, True),
    (1, 8, 33, 4097, 128, "bf16", False, 0.0, True),      # a last block of one key
    (1, 1, 2, 16384, 64, "fp16", False, 0.0, True),
    (1, 1, 31, 5000, 256, "bf16", False, 0.0, True),
    (1, 4, 300, 3000, 256, "fp16", False, 0.01, True),
    (2, 8, 1024, 1024, 128, "fp16", False, 0.0, False),  # halves
    (2, 24, 200, 1500, 64, "bf16", False, 0.0, False),
    (1, 16, 1111, 1111, 128, "bf16", True, 0.0, False),
    (2, 2, 321, 321, 64, "fp16", True, 0.0, False),
    (1, 6, 3000, 3000, 128, "fp16", True, 0.01, True),   # slices of 128-row tiles: the first Q tiles lie in one slice
    (1, 3, 1500, 1500, 64, "bf16", True, 0.0, True),
    (1, 2, 1409, 1409, 256, "fp16", True, 0.0, True),    # a last Q tile of one row
    (1, 2, 640, 640, 128, "fp16", True, 0.0, False),
    (2, 24, 665, 665, 128, "bf16", True, 0.0, False),    # halves, more Q tiles than CUs: longest first
    (6, 16, 400, 400, 256, "fp16", True, 0.0, False),
    (5, 11, 897, 897, 64, "fp16", True, 0.0, False),     # heads not a multiple of 8
]


@pytest.mark.parametrize("B,H,Nq,Nk,d,dtype,causal,outliers,sliced", CASES)
def test_split_parity(B, H, Nq, Nk, d, dtype, causal, outliers, sliced):
    print(f"split case B={B} H={H} Nq={Nq} Nk={Nk} d={d} {dtype} causal={causal}", flush=True)
    torch = torch_gpu()
    mask = fa2.FA2_MASK_CAUSAL if causal else fa2.FA2_MASK_NONE
    assert (fa2.fa2_workspace_bytes(B, H, Nq, Nk, d, mask) > 0) == sliced
    qb, kb, vb = _make(B, H, Nq, Nk, d, dtype, 31000 + Nq + Nk + d, outliers)
    scale = float(np.float32(d) ** np.float32(-0.5))
    o_ref, lse_ref = oracle.attention(*(oracle.widen(x, dtype) for x in (qb, kb, vb)), scale, causal=causal)
    o, lse = _run(qb, kb, vb, dtype, scale, causal)
    _check(o, lse, o_ref, lse_ref, "with a workspace")
    # the same problem through the C ABI without a workspace, and with one that is too small
    q, k, v = (_guarded(x, dtype)[0] for x in (qb, kb, vb))
    small = torch.full((1024,), 255, dtype=torch.uint8, device="cuda")
    for ws, n in ((None, 0), (small.data_ptr(), 512)):
        o = torch.full_like(q, float("nan"))
        lse = torch.full((B, H, Nq), float("nan"), dtype=torch.float32, device="cuda")
        rc = fa2.fa2_fwd_ws_raw(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), lse.data_ptr(), B, H, Nq, Nk, d,
                                scale, fa2.FA2_FP16 if dtype == "fp16" else fa2.FA2_BF16, mask, ws, n,
                                torch.cuda.current_stream().cuda_stream)
        assert rc == fa2.FA2_OK
        torch.cuda.synchronize()
        _check(o.double().cpu().numpy(), lse.double().cpu().numpy(), o_ref, lse_ref, "without")
    assert bool((small == 255).all())


@pytest.mark.parametrize("Nq,Nk,d", [(256, 4096, 128), (1, 4096, 128), (1100, 4096, 128)])
def test_split_on_another_stream_and_in_a_graph(Nq, Nk, d):
    # the workspace belongs to the launch stream, or to the graph's pool: bits as on the current stream
    torch = torch_gpu()
    print(f"split stream/graph Nq={Nq} Nk={Nk}", flush=True)
    assert fa2.fa2_workspace_bytes(1, 8, Nq, Nk, d) > 0
    g = torch.Generator(device="cuda").manual_seed(5)
    q, k, v = (torch.randn((1, n, 8, d), generator=g, device="cuda").half() for n in (Nq, Nk, Nk))
    ref, ref_lse = fa2.fa2_fwd(q, k, v, d ** -0.5)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    outs = []
    for _ in range(5):
        o, lse = fa2.fa2_fwd(q, k, v, d ** -0.5, out=torch.empty_like(q), lse=torch.empty_like(ref_lse), stream=side)
        outs.append((o, lse))
    torch.cuda.synchronize()
    assert all(torch.equal(o, ref) and torch.equal(x, ref_lse) for o, x in outs)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        o, lse = fa2.fa2_fwd(q, k, v, d ** -0.5)
    for _ in range(4):
        o.fill_(float("nan"))
        lse.fill_(float("nan"))
        junk = torch.full((1 << 22,), 3.0, device="cuda")   # the program's own work between replays
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(o, ref) and torch.equal(lse, ref_lse) and bool((junk == 3.0).all())


@pytest.mark.parametrize("Nq,Nk,live,d,sliced", [
    (128, 641, 40, 128, False),    # wavefronts that see masked keys only
    (100, 2000, 64, 64, True),     # ... and slices that do
    (128, 1024, 1, 128, True),
    (64, 8192, 5000, 128, True),
    (200, 4000, 64, 256, True),
])
@pytest.mark.parametrize("workspace", [True, False])
def test_keys_masked_by_the_lowest_value(Nq, Nk, live, d, sliced, workspace):
    # scaled logits of masked keys overflow fp32 (lowest bf16 * log2 e); the inputs are finite, so O and LSE are those of the
    # live keys, also where a wavefront, a half or a slice holds none
    print(f"split masked keys Nq={Nq} Nk={Nk} live={live} d={d} workspace={workspace}", flush=True)
    torch = torch_gpu()
    assert (fa2.fa2_workspace_bytes(1, 2, Nq, Nk, d) > 0) == sliced
    qb, kb, vb = _make(1, 2, Nq, Nk, d, "bf16", 9100 + Nk + d)
    qb, kb = mask_by_lowest_value(qb, kb, live, "bf16")
    o_ref, lse_ref = oracle.attention(oracle.widen(qb, "bf16"), oracle.widen(kb[:, :live].copy(), "bf16"),
                                      oracle.widen(vb[:, :live].copy(), "bf16"), 1.0)
    if workspace:
        o, lse = _run(qb, kb, vb, "bf16", 1.0)
    else:
        q, k, v = (_guarded(x, "bf16")[0] for x in (qb, kb, vb))
        ot = torch.full_like(q, float("nan"))
        lt = torch.full((1, 2, Nq), float("nan"), dtype=torch.float32, device="cuda")
        rc = fa2.fa2_fwd_qk_raw(q.data_ptr(), k.data_ptr(), v.data_ptr(), ot.data_ptr(), lt.data_ptr(), 1, 2, Nq, Nk, d, 1.0,
                                fa2.FA2_BF16, fa2.FA2_MASK_NONE, torch.cuda.current_stream().cuda_stream)
        assert rc == fa2.FA2_OK
        torch.cuda.synchronize()
        o, lse = ot.double().cpu().numpy(), lt.double().cpu().numpy()
    # one ulp of bf16 (P and O are rounded to it) of values up to max |V|
    assert np.all(np.isfinite(o)) and np.all(np.isfinite(lse))
    assert np.max(np.abs(o - o_ref)) <= 2.0 ** -7 * np.abs(oracle.widen(vb, "bf16")).max()
    assert np.max(np.abs(lse - lse_ref)) <= 1e-3


@pytest.mark.parametrize("B,H,Nq,Nk,d,causal", [
    (1, 1, 128, 1430, 64, False),    # five slices with the whole workspace; four would fit in a byte less
    (1, 16, 512, 8192, 128, False),
    (1, 6, 3000, 3000, 128, True),
    (1, 4, 300, 3000, 256, False),
    (1, 8, 1, 4096, 128, False),     # the single-query kernel
    (1, 1, 128, 8000, 64, False),    # slices of 32 rows in that many bytes; slices of 128 rows would take 540672
    (1, 2, 100, 8000, 256, False),
    (1, 2, 256, 2000, 64, False),    # a byte less: the same kernel in one slice
    (3, 1, 1024, 1024, 128, True),
])
def test_workspace_one_byte_short_and_exact(B, H, Nq, Nk, d, causal):
    # a byte less than fa2_workspace_bytes(): exactly fa2_fwd_qk, the workspace untouched; exactly that many: not a byte
    # past the end
    print(f"workspace edge B={B} H={H} Nq={Nq} Nk={Nk} d={d} causal={causal}", flush=True)
    torch = torch_gpu()
    mask = fa2.FA2_MASK_CAUSAL if causal else fa2.FA2_MASK_NONE
    need = fa2.fa2_workspace_bytes(B, H, Nq, Nk, d, mask)
    assert need > 0
    g = torch.Generator(device="cuda").manual_seed(11)
    q, k, v = (torch.randn((B, n, H, d), generator=g, device="cuda").half() for n in (Nq, Nk, Nk))
    ws = torch.empty(need + 4096, dtype=torch.uint8, device="cuda")

    def call(ws_ptr, nbytes):
        ws.fill_(0xA5)
        o = torch.full_like(q, float("nan"))
        lse = torch.full((B, H, Nq), float("nan"), dtype=torch.float32, device="cuda")
        args = (q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), lse.data_ptr(), B, H, Nq, Nk, d, d ** -0.5,
                fa2.FA2_FP16, mask)
        stream = torch.cuda.current_stream().cuda_stream
        rc = fa2.fa2_fwd_qk_raw(*args, stream) if ws_ptr is None else fa2.fa2_fwd_ws_raw(*args, ws_ptr, nbytes, stream)
        assert rc == fa2.FA2_OK
        torch.cuda.synchronize()
        return o, lse

    o_ref, lse_ref = call(None, 0)
    o, lse = call(ws.data_ptr(), need - 1)
    assert bool((ws == 0xA5).all()), "a workspace that is too small was written"
    assert torch.equal(o, o_ref) and torch.equal(lse, lse_ref)
    o, lse = call(ws.data_ptr(), need)
    assert bool((ws[need:] == 0xA5).all()) and not bool((ws[:need] == 0xA5).all())
    assert bool((o.float() - o_ref.float()).abs().max() <= 2e-3) and bool((lse - lse_ref).abs().max() <= 1e-5)


@pytest.mark.parametrize("Nq,Nk,d", [(256, 4096, 128), (1, 4096, 128), (1100, 4096, 128)])
def test_capture_begun_without_torch_holds_no_pool_memory(Nq, Nk, d):
    # nothing keeps torch's ordinary memory for such a graph: the call must leave its keys unsplit rather than take scratch
    # that other tensors own when the graph is replayed
    print(f"raw capture Nq={Nq} Nk={Nk}", flush=True)
    torch = torch_gpu()
    H = 8
    need = fa2.fa2_workspace_bytes(1, H, Nq, Nk, d)
    assert need > 0
    g = torch.Generator(device="cuda").manual_seed(6)
    q, k, v = (torch.randn((1, n, H, d), generator=g, device="cuda").half() for n in (Nq, Nk, Nk))
    ref = torch.empty_like(q)
    ref_lse = torch.empty((1, H, Nq), dtype=torch.float32, device="cuda")
    assert fa2.fa2_fwd_qk_raw(q.data_ptr(), k.data_ptr(), v.data_ptr(), ref.data_ptr(), ref_lse.data_ptr(), 1, H, Nq, Nk, d,
                              d ** -0.5, fa2.FA2_FP16, fa2.FA2_MASK_NONE,
                              torch.cuda.current_stream().cuda_stream) == fa2.FA2_OK
    o, lse = torch.empty_like(ref), torch.empty_like(ref_lse)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    fa2.fa2_fwd(q, k, v, d ** -0.5, out=o, lse=lse, stream=side)   # the side stream's pool now holds a block of that size
    torch.cuda.synchronize()
    hip = fa2.load_library()   # its dependency, the HIP runtime, resolves through it
    stream, graph, graph_exec = ctypes.c_void_p(side.cuda_stream), ctypes.c_void_p(), ctypes.c_void_p()
    thread_local_mode = 1
    assert hip.hipStreamBeginCapture(stream, thread_local_mode) == 0
    try:
        fa2.fa2_fwd(q, k, v, d ** -0.5, out=o, lse=lse, stream=side)
    finally:
        assert hip.hipStreamEndCapture(stream, ctypes.byref(graph)) == 0
    assert hip.hipGraphInstantiate(ctypes.byref(graph_exec), graph, None, None, ctypes.c_size_t(0)) == 0
    with torch.cuda.stream(side):
        junk = [torch.full((need,), 7, dtype=torch.uint8, device="cuda") for _ in range(3)]
    for _ in range(3):
        o.fill_(float("nan"))
        lse.fill_(float("nan"))
        torch.cuda.synchronize()
        assert hip.hipGraphLaunch(graph_exec, stream) == 0
        torch.cuda.synchronize()
        assert torch.equal(o, ref) and torch.equal(lse, ref_lse)
        assert all(bool((x == 7).all()) for x in junk)
    assert hip.hipGraphExecDestroy(graph_exec) == 0 and hip.hipGraphDestroy(graph) == 0
