"""Build libmaddness.so for gfx950 in-tree with hipcc (always recompiles).

Each source is compiled to an object in its own hipcc process (in parallel),
then the objects are linked into the shared library.  _calls.so, the native
marshalling of the binding's fused calls, is compiled beside them.  Kernels
are launched only from the translation unit that defines them, so no
relocatable device code is needed.
"""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SOURCES = ["csrc/kernels.hip", "csrc/fused_gather.hip", "csrc/fused_rows.hip", "csrc/tiled_accum.hip",
           "csrc/row_lanes.hip", "csrc/onehot_mfma.hip", "csrc/lut_build.hip", "csrc/lut_fit.hip", "csrc/api.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # every multiply-add is written explicitly; nothing is contracted
    "-ffp-contract=off",
    # no packed fp32 instructions anywhere
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall",
]
NOISE = "packed-fp32-ops"


def _run(cmd):
    try:
        r = subprocess.run(cmd, capture_output=True, text=True)
    except OSError as e:   # no such compiler
        return 127, str(e)
    errs = "\n".join(l for l in r.stderr.splitlines() if NOISE not in l)
    return r.returncode, errs


def _calls_cmd(out: str):
    """The host compiler's line for the native marshalling of torch calls
    (csrc/torch_calls.cpp): a CPython extension against torch's own headers."""
    import sysconfig
    import torch
    t = os.path.dirname(torch.__file__)
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wno-unknown-pragmas",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            "-isystem", os.path.join(t, "include"), "-isystem", os.path.join(t, "include", "torch", "csrc", "api", "include"),
            "-isystem", sysconfig.get_paths()["include"], os.path.join(HERE, "csrc", "torch_calls.cpp"),
            "-L", os.path.join(t, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-o", out]


def build(verbose: bool = False, jobs: int = 0) -> str:
    out = os.path.join(HERE, "libmaddness.so")
    tmp = out + ".tmp"
    inc = ["-I", os.path.join(ROOT, "include"), "-I", os.path.join(HERE, "csrc")]
    jobs = jobs or min(len(SOURCES), max(1, os.cpu_count() or 1))
    with tempfile.TemporaryDirectory(prefix="mdn_build_") as tdir:
        objs, cmds = [], []
        for s in SOURCES:
            obj = os.path.join(tdir, os.path.basename(s) + ".o")
            objs.append(obj)
            cmds.append([HIPCC, *FLAGS, *inc, "-c", os.path.join(HERE, s), "-o", obj])
        if verbose:
            for c in cmds:
                print(" ".join(c), flush=True)
        calls = os.path.join(HERE, "_calls.so")
        cmds.append(_calls_cmd(calls + ".tmp"))
        with ThreadPoolExecutor(max_workers=jobs) as ex:
            results = list(ex.map(_run, cmds))
        for (rc, errs), c in zip(results, cmds):
            if rc != 0 and c is cmds[-1]:   # the library does without it (_lib.calls)
                print(f"warning: {calls} not built, the compiler failed ({rc}) on {' '.join(c)}:\n{errs}",
                      file=sys.stderr, flush=True)
                continue
            if rc != 0:
                raise RuntimeError(f"compiler failed ({rc}) on {' '.join(c)}:\n{errs}")
            if verbose and errs.strip():
                print(errs, file=sys.stderr)
        link = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp]
        if verbose:
            print(" ".join(link), flush=True)
        rc, errs = _run(link)
        if rc != 0:
            raise RuntimeError(f"link failed ({rc}):\n{errs}")
    os.replace(tmp, out)
    if results[-1][0] == 0:
        os.replace(calls + ".tmp", calls)
    elif os.path.exists(calls):
        os.remove(calls)   # (an older one may not fit the library or torch)
    return out


if __name__ == "__main__":
    print(build(verbose=True))
