"""Compile the HIP sources of this package into ``libjetfire.so`` (gfx950 only), and the Python extension that calls it.

The library needs hipcc and nothing else.  The extension ``_native.so`` behind the Python functions also needs the headers of
this Python and of the installed torch, and belongs to that torch: build again after changing it.  Where they are missing the
library is built all the same (``python -m paper_2403_12422_amd.build --library-only``) and can be used through its C ABI.
"""
import concurrent.futures
import glob
import hashlib
import os
import re
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libjetfire.so")
EXT = os.path.join(HERE, "_native.so")
OBJ_DIR = os.path.join(HERE, "_build")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-fast-math", "-ffp-contract=off",
    # packed FP32 instructions are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # The first 14 dwords of a kernel's arguments are in registers when its waves start.  Loaded by the waves, each workgroup's first
    # request to memory waits for another one: 0.3 us of a launch.  (Attention hand-over of 8192 x 1280, four launches, 59.5 -> 58.4 us;
    # Dropout, Add, LayerNorm of the same size and their backward passes 50.2 -> 48.0.)  What a kernel needs first stands first.
    "-mllvm", "-amdgpu-kernarg-preload-count=14",
    "-Wall", "-Wno-unused-function",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def source_digest() -> str:
    """Digest of the device sources without their comments and of the compiler's flags: tells whether a recorded profile is of the present kernels."""
    h = hashlib.sha256("\n".join(HIPCC_FLAGS).encode())
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):      # .hip and .hpp
        with open(path) as f:
            code = [re.sub(r"\s+", " ", line.split("//")[0]).strip() for line in f]
        h.update("\n".join([os.path.basename(path)] + [line for line in code if line]).encode())
    return h.hexdigest()[:16]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass warns that it does not know the packed-fp32 feature; that line is noise
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("build step failed: " + cmd[0] + "\n" + out)
    if verbose and out.strip():
        print(out)


def _hipcc():
    return os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _extension_commands():
    """The host-only CPython extension (csrc/jf_python.cpp): compiled as plain C++ against torch's headers, linked to the
    library beside it: the compile and the link command."""
    import torch

    root = os.path.dirname(torch.__file__)
    inc, lib = os.path.join(root, "include"), os.path.join(root, "lib")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    obj = os.path.join(OBJ_DIR, "jf_python.o")
    compile_ = [_hipcc(), "-x", "c++", "-O2", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
                "-I", INCLUDE, "-isystem", inc, "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"),
                "-isystem", sysconfig.get_paths()["include"], "-isystem", os.path.join(rocm, "include"), "-Wall",
                "-c", os.path.join(CSRC, "jf_python.cpp"), "-o", obj]
    link = [_hipcc(), "-shared", "-fPIC", obj, "-o", EXT, "-L", HERE, "-ljetfire", "-L", lib, "-lc10",
            "-lc10_hip", "-ltorch_cpu", "-ltorch_hip", "-ltorch_python", "-Wl,-rpath,$ORIGIN"]
    return compile_, link


def build(verbose: bool = False, jobs: int = 0, extension: bool = True) -> str:
    """Always recompiles every source (one hipcc process per translation unit, in parallel), then links;
    returns the path of the shared object.  If the extension cannot be built this raises with the library in place."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    jobs = jobs or min(16, os.cpu_count() or 1)
    if os.path.exists(EXT):
        os.remove(EXT)      # it belongs to the library that it was built with
    objs = []
    with concurrent.futures.ThreadPoolExecutor(max_workers=jobs) as pool:
        futures = []
        for src in sources():
            obj = os.path.join(OBJ_DIR, os.path.basename(src)[:-4] + ".o")
            objs.append(obj)
            futures.append(pool.submit(_run, [_hipcc(), *HIPCC_FLAGS, "-I", INCLUDE, "-I", CSRC, "-c", src, "-o", obj], verbose))
        ext_object = pool.submit(_compile_extension, verbose) if extension else None
        for f in futures:
            f.result()
    _run([_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB], verbose)
    if extension:
        try:
            _run(ext_object.result(), verbose)
        except Exception as e:
            raise RuntimeError(f"{LIB} is built, the Python extension {EXT} is not (it needs the headers of Python and torch)") from e
    return LIB


def _compile_extension(verbose):
    compile_, link = _extension_commands()
    _run(compile_, verbose)
    return link


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv, extension="--library-only" not in sys.argv))
