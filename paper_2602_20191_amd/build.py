"""Builds libmbq.so (HIP, gfx950) in-tree with hipcc, and the native half of the torch binding (_mbq_torch.so, host code
against torch's headers).  Run: python -m paper_2602_20191_amd.build"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmbq.so")
TORCH_LIB = os.path.join(HERE, "_mbq_torch.so")
OBJ_DIR = os.path.join(HERE, "_build")

SOURCES = [
    # (file, extra flags)
    ("mbq_api.hip", []),
    ("mbq_encode.hip", ["-ffp-contract=off"]),   # the code recursion is specified unfused
    ("mbq_route.hip", ["-ffp-contract=off"]),
    ("mbq_act.hip", ["-ffp-contract=off"]),      # every step of the activation quantiser is one fp32 operation
    ("mbq_linear_simple.hip", []),
    ("mbq_linear_decode.hip", []),
    ("mbq_linear_decode16.hip", []),
    ("mbq_linear_mid.hip", []),
    ("mbq_linear_decode_f4.hip", []),
    ("mbq_linear_decode_f4_ws.hip", []),
    ("mbq_linear_prefill.hip", []),
    ("mbq_bench.hip", []),
]

COMMON = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from forming packed-fp32 VALU ops
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
    "-DMBQ_BUILDING=1",
]


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found")
    return exe


def _run(cmd):
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in proc.stdout.splitlines()
                    if "is not a recognized feature for this target" not in l)
    if proc.returncode != 0:
        raise RuntimeError("command failed: %s\n%s" % (" ".join(cmd), out))
    return out


def torch_command():
    import sysconfig

    import torch
    from torch.utils import cpp_extension

    includes = cpp_extension.include_paths() + [sysconfig.get_paths()["include"]]
    # NDEBUG: without it the headers' reference checks put a thread-local counter into the module.  The C library then takes
    # the slow path at every thread-local access of all libraries loaded before, from the module's import to the end of the
    # process (torch.empty 1.1 -> 1.4 us, a routing call of the binding 17.7 -> 19.7).
    return (["g++", "-O2", "-DNDEBUG", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
             "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI)] +
            [x for i in includes for x in ("-isystem", i)] + [os.path.join(CSRC, "mbq_torch.cpp"), "-o", TORCH_LIB] +
            ["-L" + p for p in cpp_extension.library_paths()] + ["-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10"])


def build(verbose: bool = False, save_temps: bool = False) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    cc = hipcc()
    objs = []
    jobs = []
    for src, extra in SOURCES:
        obj = os.path.join(OBJ_DIR, src.replace(".hip", ".o"))
        objs.append(obj)
        cmd = [cc] + COMMON + extra + ["-c", os.path.join(CSRC, src), "-o", obj]
        if save_temps:
            cmd += ["-save-temps=obj"]
        jobs.append(cmd)
    with ThreadPoolExecutor(max_workers=min(6, os.cpu_count() or 1)) as pool:
        binding = pool.submit(lambda: _run(torch_command()))
        for out in pool.map(_run, jobs):
            if verbose and out.strip():
                print(out)
        _run([cc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs)
        # the library is a C ABI that needs neither torch nor its headers: it stands whatever becomes of the binding's half
        binding.result()
    return LIB


if __name__ == "__main__":
    path = build(verbose=True, save_temps="--save-temps" in sys.argv)
    print("built", path)
