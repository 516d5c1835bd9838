"""Builds the HIP shared library in-tree for gfx950 (cross-compiles without a GPU)."""
import os
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(HERE, "libsim355.so")
SOURCES = [os.path.join(HERE, "csrc", f) for f in (
    "step_warm_pairs.hip", "step_pairs.hip", "step_plain.hip", "step_warm.hip", "step_newton_warm.hip", "step_newton.hip",
    "sim.hip")]
HEADERS = [os.path.join(HERE, "csrc", f) for f in (
    "model.hpp", "contact_gen.hpp", "step_kernel.hpp", "step_variants.hpp", "step_variants_impl.hpp", "regroup.hpp",
    "builtin_robots.hpp")] + [os.path.join(os.path.dirname(HERE), "include", "sim.h")]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed fp32 VALU forms are kept off on this target
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def is_stale():
    if not os.path.exists(LIB_PATH):
        return True
    t = os.path.getmtime(LIB_PATH)
    return any(os.path.getmtime(f) > t for f in SOURCES + HEADERS)


def build(force=True, verbose=False, extra=()):
    if not force and not is_stale():
        return LIB_PATH
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, os.path.basename(src) + ".o") for src in SOURCES]

        def compile_one(src, obj):
            cmd = [hipcc] + HIPCC_FLAGS + list(extra) + ["-c", "-o", obj, src]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True)

        # one hipcc per source, side by side (the longest first)
        with ThreadPoolExecutor(max_workers=min(len(SOURCES), os.cpu_count() or 1)) as pool:
            for done in [pool.submit(compile_one, s, o) for s, o in zip(SOURCES, objs)]:
                done.result()
        subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-o", LIB_PATH] + objs, check=True)
    return LIB_PATH


if __name__ == "__main__":
    build(force=True, verbose=True)
