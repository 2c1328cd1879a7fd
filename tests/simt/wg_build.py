"""Builds the batch and the transitive closure (batch.hip, tc_reduce.hip)
against the CPU emulation into tests/simt/_build/libllp_simt_wg.so.  The
kernels' dynamic LDS declarations are rewritten to plain arrays (wg_prelude.h);
nothing else of the sources changes.  Test infrastructure only."""
from __future__ import annotations

import os
import shutil
import subprocess

import build as base

LIB = os.path.join(base.OUT, "libllp_simt_wg.so")
DYNAMIC = {"batch.hip": "alignas(8) int lds[40960];", "tc_reduce.hip": "unsigned long long tl[20480];"}
HOST = ("llp_host.cpp", "tune.cpp", "abi.cpp")
# sizes abi.cpp asks of the sources that are not built here
STUBS = """#include <stddef.h>
#include <stdint.h>
namespace llp {
size_t sm_workspace_bytes(int64_t) { return 256; }
size_t graph_workspace_bytes(int64_t, int64_t, int) { return 256; }
size_t jobs_workspace_bytes(int64_t, int64_t, int) { return 256; }
}
"""


def build() -> str:
    os.makedirs(base.OUT, exist_ok=True)
    odir = os.path.join(base.OUT, f"wg-{os.getpid()}")
    os.makedirs(odir, exist_ok=True)
    san = ["-fsanitize=address", "-fno-omit-frame-pointer"] if base.asan_runtime() else []
    flags = ["-std=c++17", "-O1", "-g", "-fPIC", "-I", base.HERE, "-I", base.CSRC, "-Wno-unused-result",
             "-Wno-attributes", "-include", os.path.join(base.HERE, "wg_prelude.h"), *san]
    srcs = [os.path.join(base.CSRC, f) for f in HOST] + [os.path.join(base.HERE, "simt.cpp")]
    for f, array in DYNAMIC.items():
        with open(os.path.join(base.CSRC, f)) as h:
            text = h.read()
        assert text.count("extern __shared__") == 1
        text = text.replace("extern __shared__", "SIMT_DYNAMIC")
        srcs.append(os.path.join(odir, f + ".cpp"))
        with open(srcs[-1], "w") as h:
            h.write(text + f"\nnamespace llp {{ {array} }}\n")
    srcs.append(os.path.join(odir, "stubs.cpp"))
    with open(srcs[-1], "w") as h:
        h.write(STUBS)
    objs = []
    for src in srcs:
        obj = os.path.join(odir, os.path.basename(src) + ".o")
        r = subprocess.run(["g++", *flags, "-c", src, "-o", obj], capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"g++ failed for {src}:\n{r.stderr}")
        objs.append(obj)
    tmp = LIB + f".{os.getpid()}.tmp"
    r = subprocess.run(["g++", *san, "-shared", "-o", tmp, *objs], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB)
    shutil.rmtree(odir, ignore_errors=True)
    return LIB


if __name__ == "__main__":
    print(build())
