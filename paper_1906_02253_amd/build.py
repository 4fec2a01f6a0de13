"""Build libkfmi.so (HIP, gfx950) in-tree with hipcc."""
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libkfmi.so")
SOURCES = ["kf_api.hip", "kf_fit.hip", "kf_fit64.hip", "kf_find.hip", "kf_mlp.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-shared",
    "-Wall",
    "-Wno-unused-function",
    "-Wno-unknown-pragmas",
    # keep the compiler from emitting packed-FP32 VALU forms
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-fno-gpu-flush-denormals-to-zero",
]

# flags of single sources (the reason stands in the source)
SOURCE_FLAGS = {"kf_fit64.hip": ["-mllvm", "-disable-machine-licm"]}


def hipcc():
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found")


OPCOUNT_JSON = os.path.join(HERE, "opcount.json")


def build_opcount(verbose=False):
    """Compile the host operation counter of the device arithmetic and write
    its per-unit operation counts to opcount.json."""
    exe = os.path.join(HERE, "_opcount.bin")
    cmd = [hipcc(), "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-I", CSRC,
           "-o", exe, os.path.join(CSRC, "opcount.cpp")]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("hipcc failed building the operation counter")
    out = subprocess.run([exe], capture_output=True, text=True, check=True).stdout
    os.remove(exe)
    with open(OPCOUNT_JSON, "w") as f:
        f.write(out)
    return OPCOUNT_JSON


def build(verbose=False, extra=()):
    """Compiles every source to an object in parallel, then links libkfmi.so."""
    from concurrent.futures import ThreadPoolExecutor
    srcs = [os.path.join(CSRC, s) for s in SOURCES if os.path.exists(os.path.join(CSRC, s))]
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    flags = [f for f in HIPCC_FLAGS if f != "-shared"]
    objs = [os.path.join(objdir, os.path.basename(s) + ".o") for s in srcs]

    def compile_one(so):
        src, obj = so
        cmd = [hipcc(), *flags, *SOURCE_FLAGS.get(os.path.basename(src), ()), *extra, "-c", "-o", obj, src]
        if verbose:
            print(" ".join(cmd), flush=True)
        return subprocess.run(cmd, capture_output=True, text=True)

    with ThreadPoolExecutor(max_workers=len(srcs)) as ex:
        results = list(ex.map(compile_one, zip(srcs, objs)))
    for r in results:
        if r.returncode != 0:
            sys.stderr.write(r.stdout + r.stderr)
            raise RuntimeError("hipcc failed building libkfmi.so")
    tmp = LIB + ".tmp"
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("hipcc failed linking libkfmi.so")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
    print(build_opcount(verbose=True))
