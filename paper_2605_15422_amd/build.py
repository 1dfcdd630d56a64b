"""Build libdualkv.so (gfx950) in-tree with hipcc.  Usage: python -m paper_2605_15422_amd.build"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libdualkv.so")
SOURCES = ["api.hip", "fwd2.hip", "dq2.hip", "dkdv4.hip", "dkdvw.hip", "fwd256.hip", "dq256.hip", "dkdv256.hip", "dkdv512.hip", "dq512.hip", "fwd512.hip", "aux.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-munsafe-fp-atomics",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument", "-Wno-inline-asm"]

# Register allocation of the wide dK/dV kernel: its accumulators and operands fill the register file, and in the allocator's default
# order they are moved between registers (30 moves a step at head dim 128) or spilled inside the loop.  An option of the allocator is no
# part of the compiler's interface: a compiler that does not have it builds the file without.
FILE_FLAGS = {"dkdvw.hip": ["-mllvm", "-greedy-regclass-priority-trumps-globalness=1"]}


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    return "hipcc"


def build(verbose: bool = True, extra_flags=()) -> str:
    extra_flags = tuple(extra_flags) + tuple(os.environ.get("DUALKV_EXTRA_HIPCC_FLAGS", "").split())
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    hipcc = _hipcc()

    def compile_one(src):
        obj = os.path.join(objdir, src.replace(".hip", ".o"))

        def compile_with(own):
            return subprocess.run([hipcc, *FLAGS, *own, *extra_flags, "-c", os.path.join(CSRC, src), "-o", obj], capture_output=True, text=True)

        own = FILE_FLAGS.get(src, ())
        r = compile_with(own)
        if r.returncode != 0 and own and "Unknown command line argument" in r.stderr:
            print("%s: this compiler does not know %s; built without (slower, the same results)" % (src, own[-1]), file=sys.stderr)
            r = compile_with(())
        if r.returncode != 0:
            raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (src, r.stdout, r.stderr))
        if verbose and r.stderr.strip():
            lines = [ln for ln in r.stderr.splitlines() if "packed-fp32-ops" not in ln and ln.strip()]
            if lines:
                print("\n".join(lines), file=sys.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (r.stdout, r.stderr))
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build()
