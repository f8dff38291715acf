"""Build libesa.so (HIP, gfx950 only) and the Python binding's native half, _native.so, in-tree.  `python -m paper_2502_14477_amd.build`."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libesa.so")
NATIVE = os.path.join(PKG, "_native.so")

SOURCES = ["esa_api.hip", "compress.hip", "score.hip", "topk.hip", "gather.hip", "attend.hip", "attend_mfma.hip", "attend_split.hip", "rope.hip"]

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
    # a kernel's leading arguments are in scalar registers when its first wave starts: one round trip (0.3 us, measured as 640-780
    # cycles) less in front of every kernel whose arguments fit.  Steps of 5-9 kernels: 256k decode 43.9 -> 42.9 us, drafts 72.6 ->
    # 71.0, 50k tail 52.5 -> 51.7, re-encoded decode 131.6 -> 129.6.
    "-mllvm", "-amdgpu-kernarg-preload-count=14",
    # keep the compiler from forming packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Werror=unused-function",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


# per-file additions
EXTRA_FLAGS = {
    # plain v_max_f32 for the running maxima of the score sweeps (no NaN handling needed there)
    "score.hip": ["-mno-amdgpu-ieee", "-fno-honor-nans"],
}


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    raise RuntimeError("hipcc not found")


def _run(cmd):
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in p.stdout.splitlines() if "packed-fp32-ops' is not a recognized feature" not in l)
    if p.returncode != 0:
        raise RuntimeError("command failed: %s\n%s" % (" ".join(cmd), out))
    return out


def _native_flags():
    """Compiler and linker flags of the binding: host code against torch's and Python's headers."""
    import sysconfig
    from torch.utils import cpp_extension
    includes = cpp_extension.include_paths("cuda") + [sysconfig.get_paths()["include"]]
    libs = cpp_extension.library_paths("cuda")
    compile_flags = ["-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-Wall", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
                     "-I", os.path.join(ROOT, "include")] + [f for i in includes for f in ("-isystem", i)]
    link_flags = ["-shared", "-L" + PKG, "-lesa", "-Wl,-rpath,$ORIGIN"] + ["-L" + d for d in libs] + \
        ["-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python", "-lamdhip64"]
    return compile_flags, link_flags


def build(verbose: bool = False, jobs: int = 8) -> str:
    os.makedirs(OBJ, exist_ok=True)
    hipcc = _hipcc()

    def compile_one(src):
        obj = os.path.join(OBJ, src.replace(".hip", ".o"))
        out = _run([hipcc, *FLAGS, *EXTRA_FLAGS.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj])
        if verbose and out.strip():
            print(out)
        return obj

    native_compile, native_link = _native_flags()
    native_obj = os.path.join(OBJ, "binding.o")

    with ThreadPoolExecutor(max_workers=jobs) as pool:
        native = pool.submit(_run, ["g++", *native_compile, "-c", os.path.join(CSRC, "binding.cpp"), "-o", native_obj])
        objs = list(pool.map(compile_one, SOURCES))
        native.result()
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB])
    _run(["g++", native_obj, *native_link, "-o", NATIVE])
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
