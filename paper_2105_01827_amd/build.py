"""Builds the HIP library in-tree: ``python -m paper_2105_01827_amd.build``."""
import concurrent.futures
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libgala_hip.so")
SOURCES = ["gala_host.cpp", "gala_api.cpp", "gala_kernels.hip", "gala_conv_mfma.hip",
           "gala_ring1024.hip", "gala_ring2048.hip", "gala_ring4096.hip", "gala_ring8192.hip"]
HEADERS = ["gala_internal.h", "gala_ring_impl.h", "modarith.h", os.path.join("..", "..", "include", "gala.h")]
# packed-FP32 instructions are switched off for every device compile on the test machines
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-pthread", "-Wno-unused-value", "-Wno-unused-command-line-argument",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def stale():
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    return any(os.path.getmtime(os.path.join(CSRC, f)) > t for f in SOURCES + HEADERS)


def build(force=True, verbose=False):
    """Compile every source with hipcc for gfx950 into libgala_hip.so."""
    if not force and not stale():
        return LIB
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    with tempfile.TemporaryDirectory() as tmp:
        objects = [os.path.join(tmp, f + ".o") for f in SOURCES]

        def compile_one(f, obj):
            cmd = [hipcc] + FLAGS + ["-c", "-x", "hip", os.path.join(CSRC, f), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.check_call(cmd)

        with concurrent.futures.ThreadPoolExecutor(min(8, len(SOURCES))) as pool:
            list(pool.map(compile_one, SOURCES, objects))
        subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-pthread", "-o", LIB] + objects)
    return LIB


if __name__ == "__main__":
    build(force=True, verbose=True)
    print("built", LIB)
    sys.exit(0)
