"""Build libdcl.so (HIP, gfx950) in-tree with hipcc. Runs on a machine without a GPU."""
import os
import shutil
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libdcl.so")
SOURCES = ["abi.hip", "k_small.hip", "k_gemm.hip", "k_attn.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# (source, extra flags) of each object; the GEMM family's instantiations are spread over three of them
OBJECTS = [("k_gemm.hip", ["-DDCL_GEMM_PART=1"]), ("k_gemm.hip", ["-DDCL_GEMM_PART=2"]),
           ("k_gemm.hip", ["-DDCL_GEMM_PART=3"]), ("k_attn.hip", []), ("k_small.hip", []), ("abi.hip", [])]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed-FP32 instructions are kept out of generated code (all arithmetic here is scalar fp32)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unused-variable",
]


def sources():
    return [os.path.join(CSRC, s) for s in SOURCES]


def build(verbose: bool = False) -> str:
    """Compile every HIP source into libdcl.so (always recompiles). Returns the library path."""
    tmp = LIB + ".tmp%d" % os.getpid()
    objdir = tempfile.mkdtemp(prefix="dcl_build_")
    try:
        def compile_one(i):
            src, extra = OBJECTS[i]
            obj = os.path.join(objdir, "%d.o" % i)
            cmd = [HIPCC, *FLAGS, *extra, "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c",
                   os.path.join(CSRC, src), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.check_call(cmd)
            return obj
        with ThreadPoolExecutor(max_workers=min(len(OBJECTS), os.cpu_count() or 1)) as pool:
            objs = list(pool.map(compile_one, range(len(OBJECTS))))
        subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", *objs, "-o", tmp])
    finally:
        shutil.rmtree(objdir, ignore_errors=True)
    os.replace(tmp, LIB)
    return LIB


def is_stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    deps = sources() + [os.path.join(CSRC, "dcl_internal.h"), os.path.join(CSRC, "gemm_tuned.inc"),
                        os.path.join(ROOT, "include", "dcl.h")]
    return any(os.path.getmtime(p) > t for p in deps)


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
