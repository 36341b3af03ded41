"""Builds the HIP library (gfx950) in-tree, ``paper_2511_13645_amd/libfsa_hip.so``, and the binding's host
path, ``paper_2511_13645_amd/_fsa_host.*.so``."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from typing import Optional

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libfsa_hip.so")
ABI_HEADER = os.path.normpath(os.path.join(HERE, "..", "include", "fsa.h"))
SOURCES = ["fsa_api.hip", "fsa_fwd.hip", "fsa_bwd.hip", "fsa_bwd_sorted.hip", "fsa_bwd_owned.hip", "fsa_bwd_dense.hip", "fsa_wbwd.hip"]
HEADERS = ["fsa_device.hip.h", "fsa_atomic_rows.hip.h", "fsa_internal.h", "fsa_layout.h", ABI_HEADER]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-munsafe-fp-atomics",
    # keep hipcc from forming packed-fp32 instructions out of scalar float code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


HOST_SOURCE = os.path.join(HERE, "csrc_host", "fsa_host.cpp")


def host_lib() -> str:
    """Where the host path for the running Python and torch lies.  It uses parts of both that other versions lay out
    otherwise, so a build for another one has another name and is never loaded."""
    import torch
    return os.path.join(HERE, "_fsa_host.%s.torch-%s.so" % (sys.implementation.cache_tag, torch.__version__))


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    return "hipcc"


def build_hip(extra_flags=(), verbose: bool = False, out: str = LIB) -> str:
    """Compile every source to an object (side by side, one hipcc each), then link the library.
    `out` names another file for a debug build (e.g. -DFSA_TRACE), so that it never replaces the product."""
    from concurrent.futures import ThreadPoolExecutor
    import shutil
    import tempfile
    work = tempfile.mkdtemp(prefix="fsa_build_")
    try:
        def compile_one(src: str) -> str:
            obj = os.path.join(work, src + ".o")
            cmd = [hipcc(), *HIPCC_FLAGS, *extra_flags, "-c", os.path.join(CSRC, src), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True, cwd=CSRC)
            return obj
        with ThreadPoolExecutor(max_workers=min(len(SOURCES), os.cpu_count() or 1)) as pool:
            objs = list(pool.map(compile_one, SOURCES))
        tmp = out + ".tmp.%d" % os.getpid()
        cmd = [hipcc(), "--offload-arch=gfx950", "-fPIC", "-shared", "-o", tmp, *objs]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True, cwd=CSRC)
        os.replace(tmp, out)
    finally:
        shutil.rmtree(work, ignore_errors=True)
    return out


def build_host(extra_flags=(), verbose: bool = False, out: Optional[str] = None) -> str:
    """Compile the binding's host path (plain C++ against torch's headers and the CPython C API)."""
    import torch
    out = out or host_lib()
    base = os.path.dirname(torch.__file__)
    tmp = out + ".tmp.%d" % os.getpid()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           "-isystem", os.path.join(base, "include"), "-isystem", os.path.join(base, "include", "torch", "csrc", "api", "include"),
           "-isystem", sysconfig.get_paths()["include"], *extra_flags, HOST_SOURCE, "-o", tmp,
           "-L" + os.path.join(base, "lib"), "-lc10", "-ltorch_cpu", "-ltorch_python"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, out)
    return out


def is_stale() -> bool:
    if not os.path.exists(LIB) or not os.path.exists(host_lib()):
        return True
    newest = max(os.path.getmtime(os.path.join(CSRC, f)) for f in SOURCES + HEADERS)
    newest_host = max(os.path.getmtime(f) for f in (HOST_SOURCE, ABI_HEADER))
    return os.path.getmtime(LIB) < newest or os.path.getmtime(host_lib()) < newest_host


if __name__ == "__main__":
    # python -m paper_2511_13645_amd.build [--out FILE] [extra hipcc flags]; e.g. the debug build whose 2-hop
    # forward stamps per-root times (bench.py --trace-roots):  --out libfsa_hip_trace.so -DFSA_TRACE
    argv = sys.argv[1:]
    target = LIB
    if "--out" in argv:
        i = argv.index("--out")
        target = os.path.join(HERE, os.path.basename(argv[i + 1]))
        del argv[i:i + 2]
    print(build_hip(argv, verbose=True, out=target))
    if target == LIB:
        try:
            print(build_host(verbose=True))
        except (OSError, subprocess.CalledProcessError) as e:
            print("the host path was not built, the binding goes without it: %s" % e, file=sys.stderr)
