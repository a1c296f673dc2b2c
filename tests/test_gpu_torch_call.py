"""The native call of fa2_fwd against its Python path (which a given stream takes): the same bits, results and errors, whichever
form of tensors, outputs and surroundings decides between the two."""
import os
import subprocess
import sys
import sysconfig
import threading

import pytest

import paper_2312_11918_amd as fa2
from paper_2312_11918_amd import binding
from _gpu_common import torch_gpu

pytestmark = pytest.mark.gpu


def _inputs(B, H, Nq, Nk, d, dtype="float16"):
    torch = torch_gpu()
    g = torch.Generator(device="cuda").manual_seed(Nq + Nk + d)
    return [torch.randn((B, n, H, d), generator=g, device="cuda").to(getattr(torch, dtype)) for n in (Nq, Nk, Nk)]


def _native(*args):
    q, k, v, scale, out, lse, return_lse, causal = args
    return binding._load_forward()(q, k, v, scale, out, lse, return_lse, causal)


@pytest.mark.parametrize("B,H,Nq,Nk,d,dtype,causal", [
    (1, 2, 256, 256, 64, "float16", False),
    (1, 3, 100, 37, 128, "bfloat16", False),
    (2, 2, 129, 129, 256, "float16", True),
    (1, 4, 1, 4096, 128, "float16", False),      # scratch memory: keys split
    (1, 4, 200, 4096, 64, "bfloat16", False),
])
@pytest.mark.parametrize("given,return_lse", [(False, True), (True, True), (True, False), (False, False)])
def test_same_bits_as_the_python_path(B, H, Nq, Nk, d, dtype, causal, given, return_lse):
    print(f"torch call B={B} H={H} Nq={Nq} Nk={Nk} d={d} {dtype} causal={causal} given={given} lse={return_lse}", flush=True)
    torch = torch_gpu()
    q, k, v = _inputs(B, H, Nq, Nk, d, dtype)
    scale = d ** -0.5
    ref, ref_lse = fa2.fa2_fwd(q, k, v, scale, causal=causal, stream=torch.cuda.current_stream())
    out = torch.full_like(q, float("nan")) if given else None
    lse = torch.full_like(ref_lse, float("nan")) if given else None
    got = _native(q, k, v, scale, out, lse, return_lse, causal)
    assert type(got) is tuple, "not taken by the native call"
    assert got[0].dtype == q.dtype and got[0].shape == q.shape and torch.equal(got[0], ref)
    assert not given or got[0] is out
    if return_lse:
        assert torch.equal(got[1], ref_lse) and (not given or got[1] is lse)
    else:
        assert got[1] is None
    o2, l2 = fa2.fa2_fwd(q, k, v, scale, out, lse, return_lse, causal=causal)
    assert torch.equal(o2, ref) and (l2 is None) == (not return_lse)


def test_what_it_leaves_to_the_python_path():
    print("torch call: left to the Python path", flush=True)
    torch = torch_gpu()
    q, k, v = _inputs(1, 2, 128, 128, 64)
    ref, ref_lse = fa2.fa2_fwd(q, k, v, 0.125)
    rest = (0.125, None, None, True, False)

    class Sub(torch.Tensor):
        pass

    sub = q.as_subclass(Sub)
    assert _native(sub, k, v, *rest) is None
    assert torch.equal(fa2.fa2_fwd(sub, k, v, 0.125)[0], ref)
    with torch.device("cuda"):   # a torch function mode
        assert _native(q, k, v, *rest) is None
        assert torch.equal(fa2.fa2_fwd(q, k, v, 0.125)[0], ref)
    assert _native(q, k, v, "0.125", *rest[1:]) is None   # a scale that only float() reads
    assert torch.equal(fa2.fa2_fwd(q, k, v, "0.125")[0], ref)
    bad = [((q.cpu(), k, v), {}), ((q.float(), k, v), {}), ((q, k.bfloat16(), v), {}), ((q[0], k, v), {}), ((q, k, v[:, :64]), {}),
           ((q.transpose(1, 2).contiguous().transpose(1, 2), k, v), {}), ((q, k, v), {"out": q[:, :64].contiguous()}),
           ((q, k, v), {"out": torch.empty_like(q, dtype=torch.float32)}), ((q, k, v), {"lse": ref_lse.half()}),
           ((q, k, v), {"lse": ref_lse[:, :, ::2]}), ((q, k, v), {"lse": ref_lse.cpu()}), ((q, k.cpu(), v), {}), ((q, k, v.cpu()), {}),
           ((q, k, v), {"out": ref.cpu()})]
    for tensors, kw in bad:
        assert _native(*tensors, 0.125, kw.get("out"), kw.get("lse"), True, False) is None
        with pytest.raises(ValueError):
            fa2.fa2_fwd(*tensors, 0.125, **kw)
    with pytest.raises(RuntimeError):   # a tensor that a transform has wrapped has no storage
        torch.vmap(lambda x: fa2.fa2_fwd(x, k, v, 0.125)[0])(q.unsqueeze(0))


def test_refused_problems_raise_the_librarys_error():
    print("torch call: refused", flush=True)
    q, k, v = _inputs(1, 2, 128, 128, 96)
    with pytest.raises(fa2.Fa2Error) as e:
        fa2.fa2_fwd(q, k, v, 0.125)
    assert e.value.code == fa2.FA2_ERR_UNSUPPORTED
    q, k, v = _inputs(1, 2, 128, 64, 64)
    for kw, code in (({"causal": True}, fa2.FA2_ERR_UNSUPPORTED), ({}, fa2.FA2_ERR_INVALID_ARG)):
        with pytest.raises(fa2.Fa2Error) as e:
            fa2.fa2_fwd(q, k, v, 0.125 if kw else -1.0, **kw)
        assert e.value.code == code
    with pytest.raises(TypeError):
        fa2.fa2_fwd(q, k, v, None)


def test_surroundings():
    # gradients wanted, inference mode, autocast, another current stream, a graph, several threads
    print("torch call: surroundings", flush=True)
    torch = torch_gpu()
    q, k, v = _inputs(1, 2, 256, 256, 64)
    ref, ref_lse = fa2.fa2_fwd(q, k, v, 0.125)
    o, _ = fa2.fa2_fwd(q.clone().requires_grad_(), k, v, 0.125)
    assert torch.equal(o, ref) and not o.requires_grad
    with torch.inference_mode():
        assert torch.equal(fa2.fa2_fwd(q.clone(), k, v, 0.125)[0], ref)
    with torch.autocast("cuda"):
        assert torch.equal(fa2.fa2_fwd(q, k, v, 0.125)[0], ref)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        o, lse = fa2.fa2_fwd(q, k, v, 0.125)
    side.synchronize()
    assert torch.equal(o, ref) and torch.equal(lse, ref_lse)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        o, lse = fa2.fa2_fwd(q, k, v, 0.125)
    for _ in range(3):
        o.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(o, ref) and torch.equal(lse, ref_lse)
    results = [None] * 4

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            outs = [fa2.fa2_fwd(q, k, v, 0.125)[0] for _ in range(20)]
            torch.cuda.current_stream().synchronize()
            results[i] = all(torch.equal(x, ref) for x in outs)

    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert results == [True] * 4


@pytest.mark.parametrize("shape,strides", [
    ((1, 100, 2, 64), (12800, 128, 64, 1)),
    ((1, 100, 2, 64), (5, 128, 64, 1)),           # the stride of a size of one says nothing about where elements are
    ((2, 1, 4, 128), (512, 1, 128, 1)),           # ... as of one new query per sequence, cut from a channels-last tensor
    ((1, 1, 1, 64), (3, 7, 11, 1)),
])
def test_the_output_has_the_strides_of_the_query(shape, strides):
    print(f"torch call: strides {strides}", flush=True)
    torch = torch_gpu()
    q = torch.randn(12800, device="cuda").half().as_strided(shape, strides)
    k = torch.randn((shape[0], 77, *shape[2:]), device="cuda").half()
    assert q.is_contiguous()
    ref, ref_lse = fa2.fa2_fwd(q, k, k, 0.125, stream=torch.cuda.current_stream())
    assert ref.stride() == strides
    o, lse = _native(q, k, k, 0.125, None, None, True, False)
    assert o.stride() == ref.stride() and lse.stride() == ref_lse.stride()
    assert torch.equal(o, ref) and torch.equal(lse, ref_lse)


def test_allocations_that_something_watches():
    # what sees dispatched calls sees those of the Python path
    print("torch call: watched", flush=True)
    torch = torch_gpu()
    q, k, v = _inputs(1, 4, 200, 4096, 64)   # O, LSE and scratch memory
    ref = fa2.fa2_fwd(q, k, v, 0.125)[0]
    traced = torch.jit.trace(lambda *x: fa2.fa2_fwd(*x, 0.125), (q, k, v), check_trace=False)
    kinds = [n.kind() for n in traced.graph.nodes()]
    assert kinds.count("aten::empty_like") == 1 and kinds.count("aten::empty") == 1, kinds   # (no scratch: nothing returns it)
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CPU]) as profile:
        o = _native(q, k, v, 0.125, None, None, True, False)[0]
    names = [e.name for e in profile.events()]
    assert names.count("aten::empty_like") == 1 and names.count("aten::empty") == 2, names
    assert torch.equal(o, ref)


# Loaded as torch's allocator in a process of its own: whether the thread that allocates holds the interpreter's lock.
ALLOCATOR = r"""
#include <Python.h>
#include <hip/hip_runtime.h>
static int calls = 0, held = 0;
extern "C" void* counted_alloc(ssize_t size, int, hipStream_t) {
  ++calls;
  held += PyGILState_Check();
  void* p = nullptr;
  return hipMalloc(&p, (size_t)size) == hipSuccess ? p : nullptr;
}
extern "C" void counted_free(void* p, ssize_t, int, hipStream_t) { (void)hipFree(p); }
extern "C" int alloc_calls() { return calls; }
extern "C" int alloc_held() { return held; }
"""
ALLOCATING = r"""
import ctypes, sys
sys.path.insert(0, sys.argv[2])
import torch
allocator = torch.cuda.memory.CUDAPluggableAllocator(sys.argv[1], "counted_alloc", "counted_free")
torch.cuda.memory.change_current_allocator(allocator)
from paper_2312_11918_amd import binding
counts = ctypes.CDLL(sys.argv[1])
q, k, v = (torch.ones((1, n, 2, 64), device="cuda", dtype=torch.float16) for n in (512, 8192, 8192))
before = counts.alloc_calls(), counts.alloc_held()
out = binding._load_forward()(q, k, v, 0.125, None, None, True, False)   # O, LSE and scratch memory
torch.cuda.synchronize()
print("calls", counts.alloc_calls() - before[0], "held", counts.alloc_held() - before[1], "o", float(out[0].float().mean()), flush=True)
del out, q, k, v
"""


def test_other_threads_run_while_it_allocates(tmp_path):
    # memory from the driver can take long: the interpreter's lock is free meanwhile, as it is in torch's own calls
    print("torch call: allocations", flush=True)
    source, library = tmp_path / "counted.cpp", str(tmp_path / "counted.so")
    source.write_text(ALLOCATOR)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", f"-I{sysconfig.get_paths()['include']}", f"-I{rocm}/include",
                    str(source), "-o", library, f"-L{rocm}/lib", "-lamdhip64"], check=True)
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    done = subprocess.run([sys.executable, "-c", ALLOCATING, library, root], stdout=subprocess.PIPE, text=True, timeout=100)
    assert done.returncode == 0 and done.stdout.split() == ["calls", "3", "held", "0", "o", "1.0"], done
