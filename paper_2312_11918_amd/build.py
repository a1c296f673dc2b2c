"""Builds libfa2.so (the HIP kernels and their C ABI) and libfa2_probe.so (the MFMA roof probe) in-tree with hipcc
for gfx950."""
from __future__ import annotations

import os
import subprocess

_PKG = os.path.dirname(os.path.abspath(__file__))
_ROOT = os.path.dirname(_PKG)
SOURCES = [os.path.join(_PKG, "csrc", "fa2_fwd.hip")]                # the tile kernels and the C ABI
SPLIT_SOURCES = [os.path.join(_PKG, "csrc", "fa2_decode.hip"),       # one query per sequence, keys split
                 os.path.join(_PKG, "csrc", "fa2_split.hip")]        # few query tiles, keys split
STAGE_SOURCES = [os.path.join(_PKG, "csrc", "fa2_stage.hip")]        # d = 64 and 256, softmax mixed into the MFMAs
WIDE_SOURCES = [os.path.join(_PKG, "csrc", "fa2_wide.hip")]          # d = 128, partial tiles, 256 rows per workgroup
SHORT_SOURCES = [os.path.join(_PKG, "csrc", "fa2_short.hip")]        # few query rows in all
INCLUDE = os.path.join(_ROOT, "include")
LIBRARY = os.path.join(_PKG, "libfa2.so")
TORCH_SOURCE = os.path.join(_PKG, "csrc", "fa2_torch.cpp")           # the Python call on torch tensors
TORCH_LIBRARY = os.path.join(_PKG, "_fa2_torch.so")
PROBE_SOURCES = [os.path.join(_PKG, "csrc", "mfma_probe.hip")]
PROBE_LIBRARY = os.path.join(_PKG, "libfa2_probe.so")

# Packed-fp32 VALU instructions are switched off for the device pass on purpose (the host pass
# prints a harmless "unknown feature" warning).
HIPCC_FLAGS = ["-O3", "--offload-arch=gfx950", "-std=c++17", "-shared", "-fPIC",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _hipcc(sources, library, verbose):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, "-I", INCLUDE, *sources, "-o", library]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + res.stdout)
    if verbose and res.stdout.strip():
        print(res.stdout)
    return library


def build_library(verbose: bool = False) -> str:
    """Compile the HIP sources into ``libfa2.so`` and ``libfa2_probe.so`` and the call on torch tensors, which uses the
    former, into ``_fa2_torch.so``, next to this file; returns the former's path."""
    _hipcc(PROBE_SOURCES, PROBE_LIBRARY, verbose)
    _hipcc([*SOURCES, *SPLIT_SOURCES, *STAGE_SOURCES, *SHORT_SOURCES, *WIDE_SOURCES], LIBRARY, verbose)
    _build_torch_call(verbose)
    return LIBRARY


def _build_torch_call(verbose):
    import sysconfig

    import torch
    from torch.utils import cpp_extension

    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    includes = [INCLUDE, *cpp_extension.include_paths(), sysconfig.get_paths()["include"], os.path.join(rocm, "include")]
    cmd = ["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
           f'-DFA2_TORCH_VERSION="{torch.__version__}"',
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *(f"-isystem{p}" for p in includes), TORCH_SOURCE,
           "-o", TORCH_LIBRARY, f"-L{_PKG}", "-l:libfa2.so", f"-L{torch_lib}", "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_hip", "-ltorch_python",
           f"-L{os.path.join(rocm, 'lib')}", "-lamdhip64", "-Wl,-rpath,$ORIGIN"]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ failed:\n" + res.stdout)


def resource_usage(sources=SOURCES):
    """Compile the kernels of `sources` for the device only and return what the compiler reports per kernel: a list
    of dicts with the (demangled) kernel name, VGPRs, AGPRs, SGPRs, scratch bytes per lane, LDS bytes per workgroup
    and wavefronts per SIMD.  Nothing is written; used by the test that keeps every kernel free of scratch."""
    import re

    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    flags = [f for f in HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    report = ""
    for source in sources:
        cmd = [hipcc, *flags, "-I", INCLUDE, "--cuda-device-only", "-c", "-o", os.devnull,
               "-Rpass-analysis=kernel-resource-usage", source]
        res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + res.stdout)
        report += res.stdout
    keys = {"TotalSGPRs": "sgprs", "VGPRs": "vgprs", "AGPRs": "agprs", "ScratchSize [bytes/lane]": "scratch_bytes_per_lane",
            "Occupancy [waves/SIMD]": "waves_per_simd", "LDS Size [bytes/block]": "lds_bytes_per_workgroup"}
    kernels, cur = [], None
    for line in report.splitlines():
        m = re.search(r"remark:\s+(.*?)\s+\[-Rpass-analysis", line)
        if not m:
            continue
        text = m.group(1).strip()
        if text.startswith("Function Name:"):
            cur = {"mangled": text.split(":", 1)[1].strip()}
            kernels.append(cur)
        elif cur is not None and ":" in text:
            k, v = text.rsplit(":", 1)
            if k.strip() in keys:
                cur[keys[k.strip()]] = int(v)
    for k in kernels:
        m = re.search(r"fa2_fwd_kernelILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELb(\d)ELb(\d)ELb(\d)E", k["mangled"])
        if m:
            dt, d, wv, nbuf, causal, ragged, cut = (int(x) for x in m.groups())
            k["name"] = (f"fa2_fwd_kernel<{'fp16' if dt == 0 else 'bf16'}, d={d}, {wv} wavefronts, {nbuf} LDS buffers"
                         f"{', causal' if causal else ''}{', partial tiles' if ragged else ''}{', keys cut' if cut else ''}>")
            continue
        m = re.search(r"fa2_stage_kernelILi(\d+)ELi(\d+)ELb(\d)ELb(\d)E", k["mangled"])
        if m:
            k["name"] = (f"fa2_stage_kernel<{'fp16' if m[1] == '0' else 'bf16'}, d={m[2]}{', causal' if m[3] == '1' else ''}"
                         f"{', partial tiles' if m[4] == '1' else ''}>")
            continue
        m = re.search(r"fa2_short_kernelILi(\d+)ELi(\d+)ELi(\d+)ELb(\d)E", k["mangled"])
        if m:
            k["name"] = f"fa2_short_kernel<{'fp16' if m[1] == '0' else 'bf16'}, d={m[2]}, {m[3]} wavefronts{', causal' if m[4] == '1' else ''}>"
            continue
        m = re.search(r"fa2_short_merge_kernelILi(\d+)ELi(\d+)ELb(\d)E", k["mangled"])
        if m:
            k["name"] = f"fa2_short_merge_kernel<{'fp16' if m[1] == '0' else 'bf16'}, d={m[2]}{', causal' if m[3] == '1' else ''}>"
            continue
        m = re.search(r"(fa2_(?:decode|decode_merge|split_merge)_kernel)ILi(\d+)ELi(\d+)E(?:Lb(\d)E)?", k["mangled"])
        if m:
            flag = {None: "", "0": ""}.get(m[4], ", causal" if "split" in m[1] else ", keys split")
            k["name"] = f"{m[1]}<{'fp16' if m[2] == '0' else 'bf16'}, d={m[3]}{flag}>"
        else:
            k["name"] = k["mangled"]
    return kernels


if __name__ == "__main__":
    import sys

    if "--resource-usage" in sys.argv:
        rows = resource_usage([*SOURCES, *SPLIT_SOURCES, *STAGE_SOURCES, *SHORT_SOURCES, *WIDE_SOURCES])
        print("| kernel | VGPRs | AGPRs | SGPRs | scratch B/lane | LDS B/workgroup | wavefronts/SIMD |")
        print("|---|---|---|---|---|---|---|")
        for k in sorted(rows, key=lambda r: r["name"]):
            print(f"| {k['name']} | {k['vgprs']} | {k['agprs']} | {k['sgprs']} | {k['scratch_bytes_per_lane']} | "
                  f"{k['lds_bytes_per_workgroup']} | {k['waves_per_simd']} |")
    else:
        print(build_library(verbose=True))
