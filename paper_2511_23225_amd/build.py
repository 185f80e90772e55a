"""Builds libtweo_hip.so (the C-ABI library of include/tweo.h) for gfx950 with hipcc."""
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libtweo_hip.so")
SOURCES = ["api.hip", "elementwise.hip", "gemm.hip", "gemm_ring.hip", "gemm_pair.hip", "gemm_mixed.hip", "gemm_any.hip"]
HEADERS = ["kernels.h", "device_utils.h", "gemm_common.h", "gemm_defer.h", "gemm_epilogue.h", "gemm_ring.h", "finish.h", os.path.join("..", "..", "include", "tweo.h")]
# packed-fp32 code generation is switched off: the compiler must not form v_pk_*_f32
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-Xclang",
         "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall", "-Wno-unused-function", "-Wno-inline-asm"]


def is_stale():
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    deps = [os.path.join(CSRC, f) for f in SOURCES + HEADERS]
    return any(os.path.getmtime(d) > t for d in deps)


def build_library(force=True, verbose=False, extra_flags=()):
    if not force and not is_stale():
        return LIB
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    flags = FLAGS + list(extra_flags)

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        out = "\n".join(l for l in r.stdout.splitlines()
                        if "packed-fp32-ops" not in l and "unused during compilation" not in l)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + out)
        return out

    # one compiler a source, side by side (4 minutes on eight cores, one after the other 13); a source holds no device code that another calls.
    with tempfile.TemporaryDirectory() as tmp:
        objects = [os.path.join(tmp, os.path.splitext(f)[0] + ".o") for f in SOURCES]
        jobs = [[hipcc] + [f for f in flags if f != "-shared"] + ["-c", "-o", o, os.path.join(CSRC, f)]
                for f, o in zip(SOURCES, objects)]
        with ThreadPoolExecutor(max(1, min(len(jobs), int(os.environ.get("MAX_JOBS") or os.cpu_count() or 1)))) as pool:
            out = "\n".join(o for o in pool.map(run, jobs) if o.strip())
        run([hipcc, "--offload-arch=gfx950", "-fPIC", "-shared"] + list(extra_flags) + ["-o", LIB] + objects)
    if verbose and out.strip():
        print(out)
    return LIB


if __name__ == "__main__":
    build_library(verbose=True, extra_flags=sys.argv[1:])
    print("built", LIB)
