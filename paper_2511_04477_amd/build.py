"""Compile libspqt.so (and its benchmark, timeline and test variants) for gfx950 with hipcc, which
cross-compiles without a GPU.

Every source is compiled to an object of its own, several at a time, and the objects are linked;
objects live in `_build/` next to this file and are rebuilt on every call.
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libspqt.so")
SOURCES = ["pack.cpp", "quant_cb.cpp", "gather.hip", "gemv.hip", "gemv_cb.hip", "gemv_cb8.hip", "gemv_cb2.hip", "gemv_list.hip",
           "gemv_bal.hip"]
CALIB_LIB = os.path.join(PKG, "libspqt_calib.so")       # benchmark-only helper kernels
CALIB_SOURCES = ["calib.hip", "baseline_rowmajor.hip"]
# The same kernels with wall-clock stamps per wavefront (python -m paper_2511_04477_amd.timeline).
TIMELINE_LIB = os.path.join(PKG, "libspqt_timeline.so")
# The group-layout GEMV entry points with silent producers and a reducer that waits for a handful of polls only:
# what the tests use to run the give-up path of the exchange (NaN outputs, poison flag) without a stalled kernel.
GIVEUP_LIB = os.path.join(PKG, "libspqt_giveup.so")
GIVEUP_SOURCES = ["pack.cpp", "gemv.hip", "gemv_list.hip", "gemv_bal.hip"]
# The library with reducers that never wait in a block-row spread over several XCDs: they hand the sum over at once.
HANDOVER_LIB = os.path.join(PKG, "libspqt_handover.so")

# Device calls of binding.py as a Python extension module: host code against the headers of one Python and one torch.  The only part that needs
# torch; the libraries are built, and the binding works, without it.
FASTCALL_LIB = os.path.join(PKG, "_fastcall" + sysconfig.get_config_var("EXT_SUFFIX"))
FASTCALL_SOURCE = "fastcall.cpp"

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from forming packed-fp32 VALU ops
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # matrix-core results stay in ordinary VGPRs: with a separate accumulator file the kernels that use
    # v_mfma would copy their sums to scale and add them
    "-mllvm", "-amdgpu-mfma-vgpr-form",
    # the first 14 dwords of a kernel's arguments are in scalar registers when a wavefront starts (gemv_common.hpp)
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wno-unused-command-line-argument",
]
JOBS = max(1, min(8, os.cpu_count() or 1))


def _hipcc() -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    return hipcc if os.path.exists(hipcc) else "hipcc"


def _run(cmd, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    noise = "is not a recognized feature for this target"
    out = "\n".join(ln for ln in res.stdout.splitlines() if noise not in ln)
    if res.returncode != 0:
        raise RuntimeError(os.path.basename(cmd[0]) + " failed:\n" + out)
    if verbose and out.strip():
        print(out)


def _fastcall_command(lib: str):
    """The compile command of the extension module, or None without torch."""
    try:
        import torch
    except ImportError:
        return None
    base = os.path.dirname(torch.__file__)
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}",
            f'-DSPQT_TORCH_VERSION="{torch.__version__}"',
            "-isystem", os.path.join(base, "include"), "-isystem", os.path.join(base, "include/torch/csrc/api/include"), "-isystem", "/opt/rocm/include",
            "-I", sysconfig.get_paths()["include"], "-I", os.path.join(ROOT, "include"), "-o", lib, os.path.join(CSRC, FASTCALL_SOURCE),
            "-L", os.path.join(base, "lib"), "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip"]


def _jobs(lib: str, sources, defines=(), tag: str = ""):
    """(compile command, ...) per source and the link command of one library."""
    objs = [os.path.join(OBJ, f"{tag}{os.path.splitext(s)[0]}.o") for s in sources]
    common = [_hipcc(), *HIPCC_FLAGS, *[f"-D{d}" for d in defines], "-I", os.path.join(ROOT, "include"), "-I", CSRC]
    compiles = [[*common, "-c", "-o", o, os.path.join(CSRC, s)] for s, o in zip(sources, objs)]
    return compiles, (lib, objs)


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    plan = [_jobs(CALIB_LIB, CALIB_SOURCES),
            _jobs(TIMELINE_LIB, SOURCES, defines=("SPQT_TIMELINE=1",), tag="tl_"),
            _jobs(GIVEUP_LIB, GIVEUP_SOURCES, defines=("SPQT_TEST_GIVE_UP=1",), tag="gu_"),
            _jobs(HANDOVER_LIB, SOURCES, defines=("SPQT_TEST_HAND_OVER=1",), tag="ho_"),
            _jobs(LIB, SOURCES)]
    # every object of every library in one pool (longest first), then the links
    compiles = sorted((c for cs, _ in plan for c in cs), key=lambda c: -os.path.getsize(c[-1]))
    fastcall = FASTCALL_LIB + f".tmp{os.getpid()}"
    command = _fastcall_command(fastcall)
    with ThreadPoolExecutor(JOBS) as pool:
        module = pool.submit(_run, command, verbose) if command else None
        list(pool.map(lambda c: _run(c, verbose), compiles))
        for _, (lib, objs) in plan:
            tmp = lib + f".tmp{os.getpid()}"
            _run([_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs], verbose)
            os.replace(tmp, lib)
        if module:
            module.result()
            os.replace(fastcall, FASTCALL_LIB)
        else:
            print("torch is not installed: _fastcall, the quicker way of device calls, is not built", flush=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
