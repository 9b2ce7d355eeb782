"""Build libtriinv.so (hand-written HIP for gfx950) in-tree with hipcc.

One translation unit per (C, operand type) pair plus the C-ABI file, compiled in parallel and
linked into paper_2605_21325_amd/libtriinv.so.  Packed-fp32 code generation is switched off
for every device compile.  Beside it the host compiler builds the binding's native argument
handling, paper_2605_21325_amd/_fastcall.so, from Python's and torch's headers; the binding does without it
where that fails.
"""
from __future__ import annotations

import json
import os
import re
import subprocess
import sys
import sysconfig
import warnings
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libtriinv.so")
FASTCALL = os.path.join(HERE, "_fastcall.so")
RESOURCES = os.path.join(HERE, "kernel_resources.json")  # registers / scratch / LDS of every kernel, from the compiler

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wno-pass-failed", "-Wno-unused-command-line-argument",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # keep MFMA results in ordinary VGPRs: the kernels post-process every accumulator with vector
         # ALU code, and the accumulator-register form costs one copy instruction per register
         "-mllvm", "-amdgpu-mfma-vgpr-form=1",
         "-Rpass-analysis=kernel-resource-usage"]

# slowest units first so the pool stays busy
UNITS = [
    (f"inst_nb{nb}_op{op}_fwd", "inst.hip", [f"-DTRIINV_INST_NB={nb}", f"-DTRIINV_INST_OP={op}", "-DTRIINV_INST_FWD=1"])
    for nb in (8, 4, 2, 1) for op in (0, 1, 2)
] + [
    (f"inst_nb{nb}_op{op}", "inst.hip", [f"-DTRIINV_INST_NB={nb}", f"-DTRIINV_INST_OP={op}"])
    for nb in (8, 4, 2, 1) for op in (0, 1, 2)
] + [
    (f"solve_nb{nb}_op{op}", "solve.hip", [f"-DTRIINV_INST_NB={nb}", f"-DTRIINV_INST_OP={op}"])
    for nb in (8, 4, 2, 1) for op in (0, 1, 2)
] + [("api", "api.hip", [])]


def _sources_mtime() -> float:
    return max(os.path.getmtime(os.path.join(CSRC, f)) for f in os.listdir(CSRC))


_REMARK = re.compile(r"remark:\s+(Function Name|VGPRs|AGPRs|ScratchSize \[bytes/lane\]|Occupancy \[waves/SIMD\]|"
                     r"VGPRs Spill|LDS Size \[bytes/block\]): (\S+)")


def _parse_resources(stderr: str) -> dict:
    out, cur = {}, None
    for key, val in _REMARK.findall(stderr):
        if key == "Function Name":
            cur = out.setdefault(val, {})
        elif cur is not None:
            cur[{"VGPRs": "vgpr", "AGPRs": "agpr", "ScratchSize [bytes/lane]": "scratch", "Occupancy [waves/SIMD]": "occupancy",
                 "VGPRs Spill": "vgpr_spill", "LDS Size [bytes/block]": "lds"}[key]] = int(val)
    return out


def _compile(unit):
    name, src, defs = unit
    out = os.path.join(OBJ, name + ".o")
    cmd = [HIPCC, *FLAGS, *defs, "-c", os.path.join(CSRC, src), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {name}:\n{r.stderr[-4000:]}")
    return out, _parse_resources(r.stderr)


def fastcall_stamp() -> str:
    """The Python and the torch whose headers a module is built from: it reads their objects through inline functions."""
    import torch
    return f"triinv fastcall, Python {sys.hexversion:08x}, torch {torch.__version__} {torch.version.git_version}"


def build_fastcall() -> str:
    import torch
    root = os.path.dirname(torch.__file__)
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f"-I{sysconfig.get_paths()['include']}",
           f'-DTRIINV_BUILT_FOR="{fastcall_stamp()}"', f"-I{root}/include", f"-I{root}/include/torch/csrc/api/include", os.path.join(CSRC, "fastcall.cpp"), "-o", FASTCALL,
           f"-L{root}/lib", "-ltorch_python", "-ltorch_cpu", "-lc10"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed for fastcall.cpp:\n{r.stderr[-4000:]}")
    return FASTCALL


def _current(path: str) -> bool:
    return os.path.exists(path) and os.path.getmtime(path) >= _sources_mtime()


def _fastcall_current() -> bool:
    if not _current(FASTCALL):
        return False
    with open(FASTCALL, "rb") as f:
        return fastcall_stamp().encode() in f.read()


def build(force: bool = False, jobs: int = 0) -> str:
    if force or not _fastcall_current():
        try:
            build_fastcall()
        except Exception as e:  # no host compiler, no headers: slower calls, the same results
            if os.path.exists(FASTCALL):
                os.remove(FASTCALL)  # of older sources
            warnings.warn(f"the native argument handling is not built: {e}")
    if not force and _current(LIB):
        return LIB
    os.makedirs(OBJ, exist_ok=True)
    jobs = jobs or min(len(UNITS), os.cpu_count() or 4, 16)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        results = list(ex.map(_compile, UNITS))
    objs = [o for o, _ in results]
    resources = {}
    for _, res in results:
        resources.update(res)
    with open(RESOURCES, "w") as f:
        json.dump(dict(sorted(resources.items())), f, indent=0)
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr[-4000:]}")
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv))
